// Internal declarations shared by the translation units of libsdp_hip.so (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <initializer_list>

#include "sdp.h"
#include "sdp_measure.h"

namespace sdp {

// ---- per-kernel event timing (sdp_profile_*) -------------------------------------------------
bool profiling_on();
bool profiling_wants(const char* name); // on, and `name` passes the filter
void profile_begin(const char* name, hipStream_t s);
// start / stop events for a launch that records them itself (hipExtLaunchKernel); false = not timed
bool profile_launch_events(const char* name, hipEvent_t* start, hipEvent_t* stop);
void profile_end(hipStream_t s);
// what sdp_profile_launch_shape will say of the last launch under `name`, while timing is on
void profile_shape(const char* name, int tile_m, int tile_n, int group_m, int stacked);
// fp32 contractions: group_m = 0, stacked = the loop
enum F32Loop { F32_STAGED = 1, F32_WAVES = 2, F32_WAVES_ONE_STAGE = 3, F32_PIPELINED = 4, F32_SPLIT = 5, F32_SPLIT_TEAMS = 6 };

struct ProfileScope {
    hipStream_t s;
    bool on;
    ProfileScope(const char* name, hipStream_t stream) : s(stream), on(name && profiling_on() && profiling_wants(name)) {
        if (on) profile_begin(name, s);
    }
    ~ProfileScope() {
        if (on) profile_end(s);
    }
};

inline int hip_status(hipError_t e) { return e == hipSuccess ? SDP_OK : SDP_ERR_HIP; }
inline int launch_status() { return hip_status(hipGetLastError()); }

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Leading dimension of `rows` rows of `min` bf16 elements that a contraction reads from the workspace: whole 128-byte lines, so
// that the 128 bytes that a depth step takes of a row are one line and not two (5000 x 1600 outputs, 2664 deep, rows of
// 5328 / 5376 bytes: 48.1 / 40.2 us; 5328 x 1600, 5000 deep, rows of 10128 / 10112 bytes: 98.7 / 83.1 us), and an odd number of
// them, since rows 2^k bytes apart fall onto the same memory channels; unless that takes the matrix out of the MFMA
// contraction's 4 GiB.
inline int64_t line_ld(int64_t min, int64_t rows) {
    const int64_t ld = (min + 63) / 64 * 64 | 64;
    return rows * ld * 2 < ((int64_t)1 << 32) ? ld : min;
}

// memory of a caller's tensor, and whether one of `out` shares any with one of `in`
struct Extent {
    const void* p;
    size_t bytes;
};
inline bool overlap(std::initializer_list<Extent> out, std::initializer_list<Extent> in) {
    for (const Extent& o : out)
        for (const Extent& i : in) {
            const uintptr_t a = (uintptr_t)o.p, b = (uintptr_t)i.p;
            if (a < b + i.bytes && b < a + o.bytes) return true;
        }
    return false;
}

// A list of rows may be given as a list of heads: row i is then row i % width of the (i / width)-th listed head, in the
// (i / held)-th of up to three stacked matrices (Q | K | V).  Read where the rows are needed: a launch that expands the heads
// first took 3 to 4 us of each attention call.
struct HeadList {
    int width = 0;          // rows of a head; 0 = the list holds the rows themselves
    uint32_t magic = 0;     // 2^32 / width, rounded up: i / width = the upper half of i x magic for i x width < 2^32
    int held = 0x7FFFFFFF;  // rows of the listed heads
    int all = 0;            // rows of one of the stacked matrices (at most 65535 heads of 128)
};
inline HeadList head_list(int width, int held_heads, int all_heads) {
    return {width, (uint32_t)((((uint64_t)1 << 32) + width - 1) / width), held_heads * width, all_heads * width};
}
// One form for both kinds of list, without a branch: several look-ups are then in flight together.
__device__ inline int listed_row(const int32_t* list, const HeadList& h, int i) {
    if (!list) return i;
    int first = 0;
    if (i >= h.held) i -= h.held, first += h.all;
    if (i >= h.held) i -= h.held, first += h.all;
    const int w = h.width ? h.width : 1;
    const int k = h.width ? (int)__umulhi((uint32_t)i, h.magic) : i;
    return first + list[k] * w + (i - k * w);
}

// the same for a list of heads alone (width > 0)
__device__ inline int head_row(const int32_t* list, const HeadList& h, int i) {
    int first = 0;
    if (i >= h.held) i -= h.held, first += h.all;
    if (i >= h.held) i -= h.held, first += h.all;
    const int k = (int)__umulhi((uint32_t)i, h.magic);
    return first + list[k] * h.width + (i - k * h.width);
}

// ---- contraction descriptor --------------------------------------------------------------------
// C[M][N] = sum_k A(m,k) * B(k,n), fp32 accumulation, all matrices row-major.
//   A(m,k) = a_km ? A[k * lda + m] : A[ra(m) * lda + k]  (a_km: A is stored depth-major, [K][M])
//   B(k,n) = b_km ? B[rb(k) * ldb + n] : B[rb(n) * ldb + k] (b_km: B is stored depth-major, [K][N])
// rb is the identity when b_gather is null, else a lookup in an int32 table (active-neuron rows); ra likewise
// with a_gather (with a_km it applies to the columns: A[k * lda + ra(m)]).  b_km: fp32 contraction, and batched launches of
// the MFMA one, which are b_km or a_km and b_km; a_km with a_gather: the same, the latter with a_gather_chunks.
// A second operand pair (A2, B2) with the same shapes and strides is used by two of the epilogues.
enum Epilogue {
    EPI_STORE = 0,       // C[rc(m) * ldc + n] = acc      (rc: optional row scatter; rc(m) < 0 drops row m)
    EPI_DUAL_ACC = 1,    // as STORE with acc = A.B + A2.B2
    EPI_SWIGLU_FWD = 2,  // g = A.B, u = A.B2: G = g, U = u, Act = silu(g) * u, all [M][N] (ld = ldc; Act: ldc3)
    EPI_SWIGLU_BWD = 3   // da = A.B; with g = Gin[m][n], u = Uin[m][n]  (ld = ldg):
                         //   dU = da silu(g), dG = da u silu'(g), act = silu(g) u, all [M][N] (ld = ldc);
                         //   plain bf16 kernel: with cidx != null also the column-compacted copies [M][pc]
                         //   (ld = ldcc): column c of Cc / Cc2 / Cc3 is column cidx[c] of dG / dU / act
};

constexpr int kMaxBatch = 4;

struct GemmDesc {
    int M = 0, N = 0, K = 0;
    const void* A = nullptr;
    const void* A2 = nullptr;
    int64_t lda = 0;
    int a_km = 0;
    const int32_t* a_gather = nullptr;
    int a_gather_chunks = 0; // a_km: the list's entries 8 i .. 8 i + 7 are consecutive, from a multiple of 8 on
    int64_t a_rows = 0; // number of rows of the stored A (bounds the gathered row index); 0 = M
    const void* B = nullptr;
    const void* B2 = nullptr;
    int64_t ldb = 0;
    int b_km = 0;
    const int32_t* b_gather = nullptr;
    int64_t b_rows = 0; // number of rows of the stored B (bounds the gathered row index); 0 = N
    int epilogue = EPI_STORE;
    // outputs
    void* C = nullptr;  // STORE / DUAL_ACC: C.  SWIGLU_FWD: G.  SWIGLU_BWD: dG
    void* C2 = nullptr; // SWIGLU_FWD: U.  SWIGLU_BWD: dU
    void* C3 = nullptr; // SWIGLU_FWD / SWIGLU_BWD: Act
    int64_t ldc = 0;
    int64_t ldc3 = 0;   // SWIGLU_FWD: leading dimension of C3, 0 = ldc
    const int32_t* c_scatter = nullptr;
    // STORE / DUAL_ACC of a single problem: optional residual, C = acc + R[m][n] (added in fp32 before the
    // result is rounded; R is indexed like C without the row scatter; R may be C itself: an element is read
    // before it is written, by the same lane)
    const void* R = nullptr;
    int64_t ldr = 0;
    // SWIGLU_BWD inputs and optional compact copies
    const void* Gin = nullptr;
    const void* Uin = nullptr;
    int64_t ldg = 0;
    void* Cc = nullptr;
    void* Cc2 = nullptr;
    void* Cc3 = nullptr;
    int64_t ldcc = 0;
    const int32_t* cidx = nullptr;
    int pc = 0;
    // with cidx and Ct (MFMA kernel): crank[n], n < N: the number of listed columns below n if n is listed, else
    // -1 - that number (see column_ranks); spares the kernel a search of cidx per wave
    const int32_t* crank = nullptr;
    // SWIGLU_BWD, MFMA kernel only: neuron-major copies Ct / Ct2 / Ct3 of dG / dU / act, [rows][ldct] with
    // Ct[r(n)][m] = dG[m][n]; r(n) = n, or with cidx the rank of n in cidx (columns not listed are dropped).
    // With Ct set, C3 may be null (act is then not stored row-major).
    void* Ct = nullptr;
    void* Ct2 = nullptr;
    void* Ct3 = nullptr;
    int64_t ldct = 0;
    HeadList heads; // bf16: with width > 0, a_gather, b_gather and c_scatter are lists of heads
    const char* name = "gemm";
    // batched launch of up to kMaxBatch problems with the same shape, strides and scatter (the
    // weight-gradient contractions): nbatch > 0 selects Ab/Bb/Cb instead of A/B/C
    int nbatch = 0;
    const void* Ab[4] = {nullptr, nullptr, nullptr, nullptr};
    int64_t ldab[4] = {0, 0, 0, 0}; // MFMA kernel, a_km: each problem's leading dimension, 0 = lda
    const void* Bb[4] = {nullptr, nullptr, nullptr, nullptr};
    void* Cb[4] = {nullptr, nullptr, nullptr, nullptr};
    // batched launches with a_km and b_km only: optional fp32 scratch of gemm_split_ws_bytes(M, N, K, nbatch) bytes.  With it, a
    // launch that has few tiles and a deep K cuts the depth into ranges that run as extra problems, and a second
    // kernel sums the ranges' partial results (gemm_choose_ksplit decides; 1 = no cut).
    void* split_ws = nullptr;
    int ksplit = 1; // set by gemm_mfma_bf16
    // batched launches only: optional fp32 scratch of gemm_tail_ws_bytes(M, N, K, nbatch) bytes.  With it, a launch
    // whose tiles fill the CUs more than once but leave the last round partly empty cuts the depth of that last
    // round's tiles into ranges (plan_tail in sdp_gemm_mfma.hip), which a second small kernel adds up.
    void* tail_ws = nullptr;
    const char* tail_name = "dw_tail_reduce"; // profile name of that second kernel
    // SWIGLU_FWD / SWIGLU_BWD and batched launches without a depth cut, MFMA kernel: transposes that have to be done when the
    // contraction is, by extra workgroups of its launch or by one of their own before it
    const struct TransposeJob* side = nullptr;
    int nside = 0;
    const char* side_name = "transposes";
};

// tags that give each call site of the MFMA contraction its own kernel symbol
enum GemmOp { OP_GATE_UP = 0, OP_DOWN = 1, OP_DACT = 2, OP_DX = 3, OP_DW = 4, OP_DW_SPLIT = 5, OP_DW_TAIL = 6 };

// fp32 contraction on the matrix cores, any shape.
int gemm_f32(const GemmDesc& g, hipStream_t s);
// A contraction d[0] with a row-major left operand (STORE or DUAL_ACC) and one or two of equal extents with depth-major ones (STORE), all
// with depth-major right operands, none of whose outputs shares memory with an operand, as one launch.  SDP_ERR_UNSUPPORTED: not
// these; nothing was launched.
int gemm_f32_group(const GemmDesc* d, int n, const char* name, hipStream_t s);
// Plain LDS-tiled bf16 contraction, any shape: what the MFMA kernel's address ranges do not take.
int gemm_simple(const GemmDesc& g, hipStream_t s);
// bf16 MFMA contraction; returns SDP_ERR_UNSUPPORTED when the shape / alignment does not fit.
int gemm_mfma_bf16(const GemmDesc& g, hipStream_t s);
bool gemm_mfma_supported(const GemmDesc& g);
// whether a launch of g alone, a single problem with a depth-major right operand (STORE or DUAL_ACC), is one for gemm_mfma_bf16
bool gemm_reads_as_stored(const GemmDesc& g);
// x, such a problem, and w, a batched one without a depth cut, none of whose outputs shares memory with an operand, as one launch:
// the same bits as in two.  gemm_pairs: whether they are worth it, from sizes and layouts; SDP_ERR_UNSUPPORTED where they are not.
bool gemm_pairs(const GemmDesc& x, const GemmDesc& w);
int gemm_mfma_pair(const GemmDesc& x, const GemmDesc& w, const char* name, hipStream_t s);
// rows that the MFMA contraction can read depth-major: 64 of them lie within 32-bit byte offsets
inline bool gemm_depth_major_ld(int64_t ld) { return ld < (int64_t)1 << 22; }
// whether the launch of g (SWIGLU_BWD, or batched without a depth cut) would carry g.side
bool gemm_carries(const GemmDesc& g);
// depth ranges a batched launch of nbatch problems of shape M x N x K would be cut into, and the scratch that takes
int gemm_choose_ksplit(int M, int N, int K, int nbatch);
size_t gemm_split_ws_bytes(int M, int N, int K, int nbatch);
// scratch of the tail cut of a batched launch (0 when none is taken)
size_t gemm_tail_ws_bytes(int M, int N, int K, int nbatch);

// ---- attention core -----------------------------------------------------------------------------
// Causal attention of n heads of width hd over Bt sequences of S tokens, on the saved projections:
// qkv [Bt S][ldq] = Q | K | V (head i at columns i hd of each part), o / dO [Bt S][ldo], lse / delta [Bt][n][S].
struct AttnCoreDesc {
    const void* qkv = nullptr;
    int64_t ldq = 0;
    const void* o = nullptr; // backward: the forward's output
    void* o_out = nullptr;   // forward
    const void* dO = nullptr;
    int64_t ldo = 0;
    float* lse = nullptr;
    float* delta = nullptr;
    void* dqkv = nullptr;
    int Bt = 0, S = 0, n = 0, hd = 0;
};
// fp32 core, hd <= 128 (SDP_ERR_UNSUPPORTED beyond)
int attn_f32_fwd(const AttnCoreDesc& c, hipStream_t s);
int attn_f32_bwd(const AttnCoreDesc& c, hipStream_t s);

// ---- one worker's MLP / attention passes with the options the block-level calls need ----------------
// As sdp_masked_mlp_fwd / _bwd and sdp_masked_attn_fwd / _bwd after argument checks, plus:
//   residual     [T][d] or null: added to the output Y (forward) in the contraction's epilogue
//   dx_residual  [T][d] or null: added to dX likewise (the gradient that arrives over the skip connection)
//   want_dw      false: the weight gradients and everything only they need (Act, dG^T, dU^T, Act^T, copies) are left out
//   idx_k / head_idx_k null (forward masking with p = F; backward masking of heads): every neuron / head, in order
int mlp_fwd_impl(int mode, int dtype, int T, int d, int F, int p, const void* X, const void* W1, const void* W3,
                 const void* W2T, const int32_t* idx_k, void* Y, void* G_save, void* U_save, const void* residual,
                 void* ws, hipStream_t s);
int mlp_bwd_impl(int mode, int dtype, int T, int d, int F, int p, const void* X, const void* dY, const void* W1,
                 const void* W3, const void* W2T, const int32_t* idx_k, const void* G_save, const void* U_save, void* dX,
                 void* dW1, void* dW3, void* dW2T, int dw_layout, const void* dx_residual, bool want_dw, void* ws,
                 hipStream_t s);
int attn_fwd_impl(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph, const void* X, const void* Wqkv,
                  const void* WoT, const int32_t* head_idx_k, void* Y, void* QKV_save, void* O_save, float* LSE_save,
                  const void* residual, void* ws, hipStream_t s);
int attn_bwd_impl(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph, const void* X, const void* dY,
                  const void* Wqkv, const void* WoT, const int32_t* head_idx_k, const void* QKV_save, const void* O_save,
                  const float* LSE_save, void* dX, void* dWqkv, void* dWoT, int dw_layout, const void* dx_residual,
                  bool want_dw, void* ws, hipStream_t s);

// out[c][r] = in[rows ? rows[r] : r][c] for r < R, c < C: (gathered) transpose of 16-bit elements; C, ld_in and ld_out
// multiples of 8, ld_out >= R (elements R .. round_up(R, 8) - 1 of an output row become zeros), 16-byte aligned bases.
int transpose_rows(const void* in, int64_t ld_in, const int32_t* rows, int R, int C, void* out, int64_t ld_out,
                   const char* name, hipStream_t s);

// Several such transposes as one launch.
constexpr int kMaxTransposeJobs = 4;
struct TransposeJob {
    const void* in;
    void* out;
    int64_t ld_in, ld_out;
    const int32_t* rows; // optional gather of input rows
    int R, C;
    HeadList heads; // of `rows` (jobs carried by the attention core's launches only)
};
int transpose_batch(const TransposeJob* jobs, int n, const char* name, hipStream_t s);
// The same jobs prepared for a launch that carries them (sdp_transpose.h): their number of 64 x 64 tiles, or -1 when
// transpose_batch would refuse them.
struct SideJobs;
int side_jobs(const TransposeJob* jobs, int n, SideJobs* side);

// out[r][:] = in[rows ? rows[r] : r][:], R rows of C floats, both without gaps
int copy_rows_f32(const float* in, const int32_t* rows, int R, int C, float* out, const char* name, hipStream_t s);

// crank[n] for n < N from the ascending list cidx[0 .. pc): the number of listed columns below n if n is listed,
// else -1 - that number
int column_ranks(const int32_t* cidx, int pc, int N, int32_t* crank, hipStream_t s);

} // namespace sdp
