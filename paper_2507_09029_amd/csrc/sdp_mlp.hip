// One worker's masked SwiGLU MLP forward and backward (the paper's Sec. 3.1 regimes applied to the
// neuron-level masks of Sec. 3.2), expressed as a fixed sequence of contractions C = A . B^T whose
// operands are read depth-contiguous, but for the weight gradients'.
//
// With n = p and S = idx_k under forward masking, n = F and S = all neurons under backward masking:
//   forward   wt      : W2c = W2T[S]^T                       ([d][n], gather + transpose, HBM-bound)
//             gate_up : [G | U] = X . [W1 | W3][S]^T         (T x n, depth d; rows of W1, W3 gathered in
//                        the operand load)  + SwiGLU epilogue -> Act
//             down    : Y  = Act . W2c^T                     (T x d, depth n)
//   backward  wt      : W1c = W1[S]^T, W3c = W3[S]^T ([d][n])
//             dact    : dA = dY . W2T[S]^T                   (T x n, depth d; rows of W2T gathered)
//                        + SwiGLU-backward epilogue -> dG, dU, Act [T][n]; under backward masking, in the
//                        place of Act, the worker's p columns of the three transposed, dG^T, dU^T, Act^T
//                        [p][T] (neuron-major, row = rank of the neuron in idx_k)
//             dw      : dW1[S] = dG^T . X, dW3[S] = dU^T . X, dW2T[S] = Act^T . dY   (p x d, depth T),
//                        one batched launch that reads X, dY and, under forward masking, dG, dU, Act as they
//                        are stored, depth-major.  With transposed copies of all of these: two workers at
//                        T = 5000, d = 1600, p = 2664 878 us, this way 821; four at T = 8192, d = 1536,
//                        p = 2048 1843, 1759; eight under backward masking at T = 16384, d = 2048, F = 5504
//                        20.6 ms, 20.1; two at T = 1024, d = 768, p = 1024 112.3, 113.7
//             dx      : dX = dG . W1c^T + dU . W3c^T         (T x d, depth 2n)
// Under backward masking the weight-gradient contraction reads only the p kept rows: the gradient is
// computed on the worker's mask and nowhere else.  fp32 tensors take the fp32 contraction, which reads every
// operand as it is stored (the weights depth-major through the worker's list, dG, dU, Act depth-major on its
// columns): no copies, four launches (five where dX and the weight gradients are not one).  bf16 operands beyond the MFMA
// kernel's address range go through the plain kernel, which reads dG, dU, Act depth-major (and, under backward masking, their
// column-compacted copies [T][p]) and X, dY from transposed copies.
#include "sdp_internal.h"

namespace {

using namespace sdp;

size_t esize(int dtype) { return dtype == SDP_F32 ? 4 : 2; }

// Leading dimensions in the workspace.  Rows of n: Act, dG, dU [T][..], W1c, W2c, W3c [d][..] (fp32 reads them as they come).
int64_t ld_neurons(int dtype, int T, int d, int n) { return dtype == SDP_BF16 ? line_ld(n, T > d ? T : d) : n; }
// Token-contiguous dG^T, dU^T, Act^T [p][T] (backward masking) and X^T, dY^T [d][T] (plain weight gradients; the same room takes
// copies of X and dY where a gradient overwrites them): 64 elements more, so that consecutive rows do not sit a power of two
// apart (rows 2^k bytes apart fall onto the same memory channels, and a depth step touches one 128-byte piece of each of
// 192-256 rows).
int64_t ld_tokens(int T, int d, int p) { return line_ld((int64_t)T + 64, d > p ? d : p); }

int check_common(int mode, int dtype, int T, int d, int F, int p) {
    if (mode != SDP_MASK_FORWARD && mode != SDP_MASK_BACKWARD) return SDP_ERR_INVALID_ARG;
    if (dtype != SDP_F32 && dtype != SDP_BF16) return SDP_ERR_INVALID_ARG;
    if (T < 1 || d < 1 || F < 1) return SDP_ERR_INVALID_ARG;
    if (p < 1 || p > F) return SDP_ERR_SHAPE;
    if ((int64_t)T * F >= ((int64_t)1 << 40)) return SDP_ERR_SHAPE;
    if (dtype == SDP_BF16 && (d % 8 || F % 8 || p % 8)) return SDP_ERR_SHAPE;
    return SDP_OK;
}

// first position of the ascending list whose entry is not below n, by all 64 lanes: a step reads 64 entries at equal distances and
// keeps the piece between two of them, so that a list of 4096 takes two dependent loads and the longest five
__device__ int lower_bound_wave(const int32_t* __restrict__ cidx, int pc, int n) {
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = pc;
    while (lo < hi) {
        const int step = (hi - lo + 63) >> 6, at = lo + lane * step;
        const int below = __popcll(__ballot(at < hi && cidx[at < hi ? at : lo] < n));
        const int end = below * (int64_t)step < hi - lo ? lo + below * step : hi;
        if (below) lo += (below - 1) * step + 1;
        hi = below ? end : lo;
    }
    return lo;
}

// Latency bounds it: a search for each column is a chain of log2(pc) loads from the L2.  So a wave finds where the entries of its 256
// columns begin and another where they end, and the columns search that piece, at most 256 entries of a list without repeats, in the LDS.
// Backward passes with backward masking, every column searching the list / this, us: T = 1024, d = 512, F = 2048, p = 1280 35.7 / 35.0,
// T = 512, d = 768, F = 2048, p = 1536 31.3 / 30.8, T = 136, d = 2048, F = 5504, p = 4128 85.0 / 84.1.
__global__ __launch_bounds__(256) void column_ranks_kernel(const int32_t* __restrict__ cidx, int pc, int N,
                                                           int32_t* __restrict__ crank) {
    __shared__ int ends[2];
    __shared__ int32_t piece[256];
    const int tid = threadIdx.x, n0 = blockIdx.x * 256, n = n0 + tid;
    if (tid < 128) {
        const int r = lower_bound_wave(cidx, pc, tid < 64 ? n0 : n0 > N - 256 ? N : n0 + 256);
        if ((tid & 63) == 0) ends[tid >> 6] = r;
    }
    __syncthreads();
    const int begin = ends[0];
    int lo = begin, hi = ends[1];
    const bool staged = hi - lo <= 256;
    if (staged && tid < hi - lo) piece[tid] = cidx[lo + tid];
    __syncthreads();
    if (n >= N) return;
    const int stop = hi;
    auto entry = [&](int i) { return staged ? piece[i - begin] : cidx[i]; };
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (entry(mid) < n) lo = mid + 1; else hi = mid;
    }
    crank[n] = lo < stop && entry(lo) == n ? lo : -1 - lo;
}

int run(int dtype, const GemmDesc& g, hipStream_t s) {
    if (dtype == SDP_F32) return gemm_f32(g, s);
    if (gemm_mfma_supported(g)) return gemm_mfma_bf16(g, s);
    if (g.nside > 0) {
        const int rc = transpose_batch(g.side, g.nside, g.side_name, s);
        if (rc != SDP_OK) return rc;
    }
    return gemm_simple(g, s);
}

} // namespace

int sdp::column_ranks(const int32_t* cidx, int pc, int N, int32_t* crank, hipStream_t s) {
    if (!cidx || !crank || pc < 0 || N < 1) return SDP_ERR_INVALID_ARG;
    ProfileScope ps("mlp_column_ranks", s);
    column_ranks_kernel<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(cidx, pc, N, crank);
    return launch_status();
}

extern "C" size_t sdp_masked_mlp_fwd_workspace_bytes(int mode, int dtype, int T, int d, int F, int p) {
    if (check_common(mode, dtype, T, d, F, mode == SDP_MASK_BACKWARD ? F : p) != SDP_OK) return 0;
    const size_t n = mode == SDP_MASK_FORWARD ? p : F;
    const size_t row_b = ld_neurons(dtype, T, d, (int)n) * esize(dtype);
    return round_up(T * row_b, 256) + round_up(d * row_b, 256);
}

extern "C" size_t sdp_masked_mlp_bwd_workspace_bytes(int mode, int dtype, int T, int d, int F, int p) {
    if (check_common(mode, dtype, T, d, F, p) != SDP_OK) return 0;
    const size_t n = mode == SDP_MASK_FORWARD ? p : F;
    const size_t e = esize(dtype);
    const int64_t ldt = ld_tokens(T, d, p);
    const size_t row_b = ld_neurons(dtype, T, d, (int)n) * e;
    size_t bytes = 3 * round_up(T * row_b, 256) + 2 * round_up(d * row_b, 256) +
                   2 * round_up((size_t)d * ldt * e, 256);
    if (mode == SDP_MASK_BACKWARD) {
        bytes += 3 * round_up((size_t)T * p * e, 256);
        bytes += 3 * round_up((size_t)p * ldt * e, 256); // neuron-major copies of dG, dU, Act on the mask
        bytes += round_up((size_t)F * sizeof(int32_t), 256); // rank of every neuron in the list
    }
    if (dtype == SDP_BF16) bytes += round_up(gemm_tail_ws_bytes(p, d, T, 3), 256); // depth ranges of the weight gradients' last round
    return bytes;
}

extern "C" int sdp_masked_mlp_fwd(int mode, int dtype, int T, int d, int F, int p, const void* X, const void* W1,
                                  const void* W3, const void* W2T, const int32_t* idx_k, void* Y, void* G_save,
                                  void* U_save, void* ws, size_t ws_bytes, void* stream) {
    if (mode == SDP_MASK_BACKWARD) p = F;
    int rc = check_common(mode, dtype, T, d, F, p);
    if (rc != SDP_OK) return rc;
    if (!X || !W1 || !W3 || !W2T || !Y || !G_save || !U_save) return SDP_ERR_INVALID_ARG;
    if (mode == SDP_MASK_FORWARD && !idx_k) return SDP_ERR_INVALID_ARG;
    for (const void* q : {X, W1, W3, W2T, (const void*)Y, (const void*)G_save, (const void*)U_save})
        if (!aligned16(q)) return SDP_ERR_INVALID_ARG;
    if (!ws || !aligned16(ws) || ws_bytes < sdp_masked_mlp_fwd_workspace_bytes(mode, dtype, T, d, F, p))
        return SDP_ERR_WORKSPACE;
    return mlp_fwd_impl(mode, dtype, T, d, F, p, X, W1, W3, W2T, idx_k, Y, G_save, U_save, nullptr, ws,
                        (hipStream_t)stream);
}

int sdp::mlp_fwd_impl(int mode, int dtype, int T, int d, int F, int p, const void* X, const void* W1, const void* W3,
                      const void* W2T, const int32_t* idx_k, void* Y, void* G_save, void* U_save, const void* residual,
                      void* ws, hipStream_t s) {
    if (mode == SDP_MASK_BACKWARD) p = F;
    int rc;
    const int n = mode == SDP_MASK_FORWARD ? p : F;
    const int32_t* gather = mode == SDP_MASK_FORWARD ? idx_k : nullptr;
    const size_t e = esize(dtype);
    char* w = (char*)ws;
    void* Act = w;
    const int64_t ldn = ld_neurons(dtype, T, d, n);
    void* W2c = w + round_up((size_t)T * ldn * e, 256);

    // The down projection reads W2: bf16 its transpose W2c, made beside gate_up, which does not need it; fp32 W2T itself.
    // An output that takes W2T's place is written too early for that: W2c is then made first (fp32: W2T's rows).
    const size_t out_b = (size_t)T * n * e, w2_b = (size_t)F * d * e;
    const TransposeJob wt{W2T, W2c, d, ldn, gather, n, d};
    const bool w2_first = dtype == SDP_F32 ? overlap({{Y, (size_t)T * d * e}, {G_save, out_b}, {U_save, out_b}}, {{W2T, w2_b}})
                                           : overlap({{G_save, out_b}, {U_save, out_b}}, {{W2T, w2_b}});
    GemmDesc dn;
    dn.name = "mlp_down";
    dn.M = T, dn.N = d, dn.K = n;
    dn.A = Act, dn.lda = ldn;
    dn.epilogue = EPI_STORE;
    dn.C = Y, dn.ldc = d;
    dn.R = residual, dn.ldr = d;
    // W2T itself, depth-major: fp32 (no output may take its place), and bf16 where the contraction takes it so
    GemmDesc as_stored = dn;
    as_stored.B = W2T, as_stored.ldb = d, as_stored.b_km = 1, as_stored.b_gather = gather, as_stored.b_rows = F;
    const bool stored = dtype == SDP_F32 ? !w2_first
                                         : !overlap({{Y, (size_t)T * d * e}, {G_save, out_b}, {U_save, out_b}}, {{W2T, w2_b}}) && gemm_reads_as_stored(as_stored);
    if (w2_first) {
        rc = dtype == SDP_F32 ? copy_rows_f32((const float*)W2T, gather, n, d, (float*)W2c, "mlp_wt_fwd", s)
                              : transpose_batch(&wt, 1, "mlp_wt_fwd", s);
        if (rc != SDP_OK) return rc;
    }
    GemmDesc gu;
    gu.name = "mlp_gate_up";
    gu.M = T, gu.N = n, gu.K = d;
    gu.A = X, gu.lda = d;
    gu.B = W1, gu.B2 = W3, gu.ldb = d, gu.b_gather = gather, gu.b_rows = F;
    gu.epilogue = EPI_SWIGLU_FWD;
    gu.C = G_save, gu.C2 = U_save, gu.ldc = n, gu.C3 = Act, gu.ldc3 = ldn;
    if (dtype == SDP_BF16 && !w2_first && !stored) gu.side = &wt, gu.nside = 1, gu.side_name = "mlp_wt_fwd";
    rc = run(dtype, gu, s);
    if (rc != SDP_OK) return rc;

    if (stored) return run(dtype, as_stored, s);
    dn.B = W2c, dn.ldb = ldn;
    if (dtype == SDP_F32) dn.ldb = d, dn.b_km = 1, dn.b_rows = n;
    return run(dtype, dn, s);
}

extern "C" int sdp_masked_mlp_bwd(int mode, int dtype, int T, int d, int F, int p, const void* X, const void* dY,
                                  const void* W1, const void* W3, const void* W2T, const int32_t* idx_k,
                                  const void* G_save, const void* U_save, void* dX, void* dW1, void* dW3, void* dW2T,
                                  int dw_layout, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_common(mode, dtype, T, d, F, p);
    if (rc != SDP_OK) return rc;
    if (dtype == SDP_BF16 && T % 8) return SDP_ERR_SHAPE;
    if (dw_layout != SDP_DW_COMPACT && dw_layout != SDP_DW_SCATTER) return SDP_ERR_INVALID_ARG;
    if (!X || !dY || !W1 || !W3 || !W2T || !idx_k || !G_save || !U_save || !dX || !dW1 || !dW3 || !dW2T)
        return SDP_ERR_INVALID_ARG;
    for (const void* q : {X, dY, W1, W3, W2T, G_save, U_save, (const void*)dX, (const void*)dW1, (const void*)dW3,
                          (const void*)dW2T})
        if (!aligned16(q)) return SDP_ERR_INVALID_ARG;
    if (!ws || !aligned16(ws) || ws_bytes < sdp_masked_mlp_bwd_workspace_bytes(mode, dtype, T, d, F, p))
        return SDP_ERR_WORKSPACE;
    return mlp_bwd_impl(mode, dtype, T, d, F, p, X, dY, W1, W3, W2T, idx_k, G_save, U_save, dX, dW1, dW3, dW2T, dw_layout,
                        nullptr, true, ws, (hipStream_t)stream);
}

int sdp::mlp_bwd_impl(int mode, int dtype, int T, int d, int F, int p, const void* X, const void* dY, const void* W1,
                      const void* W3, const void* W2T, const int32_t* idx_k, const void* G_save, const void* U_save,
                      void* dX, void* dW1, void* dW3, void* dW2T, int dw_layout, const void* dx_residual, bool want_dw,
                      void* ws, hipStream_t s) {
    int rc;
    const int n = mode == SDP_MASK_FORWARD ? p : F;
    const int32_t* gather = mode == SDP_MASK_FORWARD ? idx_k : nullptr;
    const size_t e = esize(dtype);
    const int64_t ldn = ld_neurons(dtype, T, d, n), ldt = ld_tokens(T, d, p);
    const size_t act_b = round_up((size_t)T * ldn * e, 256), wt_b = round_up((size_t)d * ldn * e, 256);
    const size_t xt_b = round_up((size_t)d * ldt * e, 256), cmp_b = round_up((size_t)T * p * e, 256);
    char* w = (char*)ws;
    void *dG = w, *dU = w + act_b, *Act = w + 2 * act_b;
    w += 3 * act_b;
    void *W1c = w, *W3c = w + wt_b;
    w += 2 * wt_b;
    void *XT = w, *dYT = w + xt_b;
    w += 2 * xt_b;
    void *dGc = dG, *dUc = dU, *Actc = Act; // forward masking: the tensors are compact already
    if (mode == SDP_MASK_BACKWARD) {
        dGc = w, dUc = w + cmp_b, Actc = w + 2 * cmp_b;
        w += 3 * cmp_b;
    }
    const size_t nm_b = round_up((size_t)p * ldt * e, 256);
    void *dGn = w, *dUn = w + nm_b, *Actn = w + 2 * nm_b; // backward masking: [p][T(+pad)], neuron-major
    if (mode == SDP_MASK_BACKWARD) w += 3 * nm_b;
    int32_t* ranks = (int32_t*)w; // backward masking: [F]
    if (mode == SDP_MASK_BACKWARD) w += round_up((size_t)F * sizeof(int32_t), 256);
    void* tail_ws = dtype == SDP_BF16 && gemm_tail_ws_bytes(p, d, T, 3) > 0 ? w : nullptr;

    if (dtype == SDP_F32) {
        GemmDesc da;
        da.name = "mlp_dact";
        da.M = T, da.N = n, da.K = d;
        da.A = dY, da.lda = d;
        da.B = W2T, da.ldb = d, da.b_gather = gather, da.b_rows = F;
        da.epilogue = EPI_SWIGLU_BWD;
        da.Gin = G_save, da.Uin = U_save, da.ldg = n;
        da.C = dG, da.C2 = dU, da.C3 = Act, da.ldc = n;
        rc = gemm_f32(da, s);
        if (rc != SDP_OK) return rc;
        // dX and the weight gradients read X, dY, W1 and W3 as they are.  Where an output takes the place of one of these (dX
        // over dY, a gradient over its weights), they read copies.
        const size_t tok_b = (size_t)T * d * e, w_b = (size_t)F * d * e;
        const size_t dw_b = (size_t)(dw_layout == SDP_DW_SCATTER ? F : p) * d * e;
        const Extent x{X, tok_b}, dy{dY, tok_b}, w1{W1, w_b}, w3{W3, w_b}, ox{dX, tok_b};
        if (want_dw ? overlap({ox, {dW1, dw_b}, {dW3, dw_b}, {dW2T, dw_b}}, {x, dy, w1, w3}) : overlap({ox}, {w1, w3})) {
            const struct { const void* in; const int32_t* rows; int R; void* out; } copies[4] = {
                {W1, gather, n, W1c}, {W3, gather, n, W3c}, {X, nullptr, T, XT}, {dY, nullptr, T, dYT}};
            for (int i = 0; i < (want_dw ? 4 : 2); ++i) {
                rc = copy_rows_f32((const float*)copies[i].in, copies[i].rows, copies[i].R, d, (float*)copies[i].out, "mlp_copy_bwd", s);
                if (rc != SDP_OK) return rc;
            }
            if (want_dw && dx_residual == dY) dx_residual = dYT;
            W1 = W1c, W3 = W3c, X = XT, dY = dYT, gather = nullptr;
        }
        GemmDesc both[2];
        GemmDesc &dx = both[0], &dw = both[1];
        dx.name = "mlp_dx";
        dx.M = T, dx.N = d, dx.K = n;
        dx.A = dG, dx.A2 = dU, dx.lda = n;
        dx.B = W1, dx.B2 = W3, dx.ldb = d, dx.b_km = 1, dx.b_gather = gather, dx.b_rows = gather ? F : n;
        dx.epilogue = EPI_DUAL_ACC;
        dx.C = dX, dx.ldc = d;
        dx.R = dx_residual, dx.ldr = d;
        if (!want_dw) return gemm_f32(dx, s);
        dw.name = "mlp_dw";
        dw.M = p, dw.N = d, dw.K = T;
        dw.lda = n, dw.a_km = 1;
        if (mode == SDP_MASK_BACKWARD) dw.a_gather = idx_k, dw.a_rows = n;
        dw.ldb = d, dw.b_km = 1;
        dw.epilogue = EPI_STORE;
        dw.ldc = d;
        dw.c_scatter = dw_layout == SDP_DW_SCATTER ? idx_k : nullptr;
        dw.nbatch = 3;
        dw.Ab[0] = dG, dw.Ab[1] = dU, dw.Ab[2] = Act;
        dw.Bb[0] = X, dw.Bb[1] = X, dw.Bb[2] = dY;
        dw.Cb[0] = dW1, dw.Cb[1] = dW3, dw.Cb[2] = dW2T;
        rc = gemm_f32_group(both, 2, "mlp_dx_dw", s);
        if (rc != SDP_ERR_UNSUPPORTED) return rc;
        rc = gemm_f32(dw, s);
        return rc != SDP_OK ? rc : gemm_f32(dx, s);
    }

    // The weight gradients read X and dY as they are (depth-major), and so they read dG, dU and Act under forward masking; under
    // backward masking dact also writes the worker's p columns of these three neuron-major.
    GemmDesc dw;
    dw.name = "mlp_dw";
    dw.M = p, dw.N = d, dw.K = T;
    dw.ldb = d, dw.b_km = 1;
    dw.epilogue = EPI_STORE;
    dw.ldc = d;
    dw.c_scatter = dw_layout == SDP_DW_SCATTER ? idx_k : nullptr;
    dw.nbatch = 3;
    if (mode == SDP_MASK_BACKWARD) {
        dw.lda = ldt;
        dw.Ab[0] = dGn, dw.Ab[1] = dUn, dw.Ab[2] = Actn;
    } else {
        dw.lda = ldn, dw.a_km = 1;
        dw.Ab[0] = dG, dw.Ab[1] = dU, dw.Ab[2] = Act;
    }
    dw.Bb[0] = X, dw.Bb[1] = X, dw.Bb[2] = dY;
    dw.Cb[0] = dW1, dw.Cb[1] = dW3, dw.Cb[2] = dW2T;
    dw.tail_ws = tail_ws, dw.tail_name = "mlp_dw_reduce";

    GemmDesc da;
    da.name = "mlp_dact";
    da.M = T, da.N = n, da.K = d;
    da.A = dY, da.lda = d;
    da.B = W2T, da.ldb = d, da.b_gather = gather, da.b_rows = F;
    da.epilogue = EPI_SWIGLU_BWD;
    da.Gin = G_save, da.Uin = U_save, da.ldg = n;
    da.C = dG, da.C2 = dU, da.ldc = ldn;
    if (want_dw && mode == SDP_MASK_FORWARD) da.C3 = Act;
    // backward masking: the epilogue also writes dG, dU and act of the worker's p columns transposed (neuron-major [p][T]),
    // in which layout the weight-gradient launch reads them depth-contiguous; act is not stored row-major
    if (want_dw && mode == SDP_MASK_BACKWARD) {
        da.Ct = dGn, da.Ct2 = dUn, da.Ct3 = Actn, da.ldct = ldt;
        da.cidx = idx_k, da.pc = p, da.crank = ranks;
    }
    const bool fused = want_dw && p % 8 == 0 && T % 8 == 0 && gemm_mfma_supported(dw) && gemm_mfma_supported(da);
    if (!fused) {
        da.Ct = da.Ct2 = da.Ct3 = nullptr, da.cidx = nullptr, da.pc = 0, da.crank = nullptr;
        // without weight gradients nothing reads act: the MFMA kernel then skips its store, the plain one writes it anyway
        if (want_dw || !gemm_mfma_supported(da)) da.C3 = Act;
        if (mode == SDP_MASK_BACKWARD && want_dw) {
            da.Cc = dGc, da.Cc2 = dUc, da.Cc3 = Actc, da.ldcc = p;
            da.cidx = idx_k, da.pc = p;
        }
    }
    // a gradient in the place of X or dY: the launch reads copies of those
    const size_t dw_b = (size_t)(dw_layout == SDP_DW_SCATTER ? F : p) * d * e, tok_b = (size_t)T * d * e;
    if (fused && overlap({{dW1, dw_b}, {dW3, dw_b}, {dW2T, dw_b}}, {{X, tok_b}, {dY, tok_b}})) {
        for (int i = 0; i < 2; ++i) { // d % 8 == 0: rows of bf16 as rows of half as many floats
            rc = copy_rows_f32((const float*)(i ? dY : X), nullptr, T, d / 2, (float*)(i ? dYT : XT), "mlp_copy_bwd", s);
            if (rc != SDP_OK) return rc;
        }
        dw.Bb[0] = dw.Bb[1] = XT, dw.Bb[2] = dYT;
        if (dx_residual == dY) dx_residual = dYT;
    }
    if (fused && mode == SDP_MASK_BACKWARD) {
        rc = column_ranks(idx_k, p, F, ranks, s);
        if (rc != SDP_OK) return rc;
    }
    // dX reads W1 and W3 as they are stored where the contraction takes them so and no output takes their place
    GemmDesc dx;
    dx.name = "mlp_dx";
    dx.M = T, dx.N = d, dx.K = n;
    dx.A = dG, dx.A2 = dU, dx.lda = ldn;
    dx.epilogue = EPI_DUAL_ACC;
    dx.C = dX, dx.ldc = d;
    dx.R = dx_residual, dx.ldr = d;
    GemmDesc as_stored = dx;
    as_stored.B = W1, as_stored.B2 = W3, as_stored.ldb = d, as_stored.b_km = 1, as_stored.b_gather = gather, as_stored.b_rows = F;
    const size_t w_b = (size_t)F * d * e, out_b = want_dw ? dw_b : 0;
    const bool apart = !overlap({{dX, tok_b}, {dW1, out_b}, {dW3, out_b}, {dW2T, out_b}}, {{W1, w_b}, {W3, w_b}});
    // and in the launch of the weight gradients, where dX does not take the place of what those read
    const bool pair = fused && apart && !overlap({{dX, tok_b}}, {{X, tok_b}, {dY, tok_b}}) && gemm_pairs(as_stored, dw);
    // otherwise the operand copies that dX and the plain weight gradients read, made beside dact, which needs none of them, or beside the
    // weight gradients where dact's tiles leave no CU idle
    const TransposeJob tj[4] = {{W1, W1c, d, ldn, gather, n, d},
                                {W3, W3c, d, ldn, gather, n, d},
                                {X, XT, d, ldt, nullptr, T, d},
                                {dY, dYT, d, ldt, nullptr, T, d}};
    const bool beside_dw = fused && !overlap({{dW1, dw_b}, {dW3, dw_b}, {dW2T, dw_b}}, {{W1, w_b}, {W3, w_b}});
    auto carried = [&] {
        GemmDesc a = da, b = dw;
        a.side = b.side = tj, a.nside = want_dw && !fused ? 4 : 2, b.nside = 2;
        return gemm_carries(a) || (beside_dw && gemm_carries(b));
    };
    // In a launch of its own dX reads the weights as stored where their copies would need a launch, and with few tokens, whose launches
    // the copies lengthen: they move 8 n d bytes beside 2 T n d flops.  Backward passes, copies / as stored, us, forward masking: own
    // launch T = 1024, d = 1600, n = 2048 79.0 / 73.8, T = 256, d = 2048, n = 4096 75.4 / 66.5 (74 shapes 12 % less, none 1 % more); carried
    // T = 512, d = 1600, n = 1024 34.1 / 32.4, T = 128, d = 2048, n = 1024 32.3 / 29.1; but T = 1024, d = 1024, n = 4096 71.6 / 74.7,
    // T = 2048, d = 768, n = 2048 67.8 / 69.2, T = 2048, d = 1024, n = 4096 130.0 / 135.3.
    const bool stored = pair || (apart && gemm_reads_as_stored(as_stored) && (T <= 512 || !carried()));
    const int first = stored ? 2 : 0;
    da.side = tj + first, da.nside = (want_dw && !fused ? 4 : 2) - first, da.side_name = "mlp_tr_bwd";
    if (beside_dw && !stored) {
        dw.side = tj, dw.nside = 2, dw.side_name = "mlp_tr_bwd";
        if (gemm_carries(da) || !gemm_carries(dw)) dw.nside = 0; else da.nside = 0;
    }
    rc = run(dtype, da, s);
    if (rc != SDP_OK) return rc;

    if (pair) return gemm_mfma_pair(as_stored, dw, "mlp_dx_dw", s);
    if (fused) {
        rc = gemm_mfma_bf16(dw, s);
        if (rc != SDP_OK) return rc;
    }
    dx.B = W1c, dx.B2 = W3c, dx.ldb = ldn;
    rc = run(dtype, stored ? as_stored : dx, s);
    if (rc != SDP_OK) return rc;

    if (fused || !want_dw) return SDP_OK;
    // plain path: the left operands depth-major ([T][ldn], or the compact copies [T][p]) as they are, the right ones transposed
    const void* lhs[3] = {dGc, dUc, Actc};
    const void* rhs[3] = {XT, XT, dYT};
    dw.nbatch = 0;
    dw.lda = mode == SDP_MASK_BACKWARD ? p : ldn, dw.a_km = 1;
    dw.ldb = ldt, dw.b_km = 0;
    for (int i = 0; i < 3; ++i) {
        dw.A = lhs[i], dw.B = rhs[i], dw.C = dw.Cb[i];
        rc = gemm_simple(dw, s);
        if (rc != SDP_OK) return rc;
    }
    return SDP_OK;
}
