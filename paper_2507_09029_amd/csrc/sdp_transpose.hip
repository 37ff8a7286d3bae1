// (Gathered) matrix transpose: out[c][r] = in[rows[r]][c].  HBM-bound helper of the bf16 contractions that read both operands
// along the depth: a worker's weights for down and dX (W2T[S]^T, W1[S]^T, W3[S]^T, each [d][n]; WoT[S]^T and Wqkv[S]^T of the
// attention block), and the token-contiguous copies that the plain weight gradients read (the MFMA ones take their operands
// as they are stored).
//
// 16-bit elements; 64 x 64 element tiles through LDS (padded rows), 256 threads (sdp_transpose.h).  Bytes moved: R*C
// element reads + R*C element writes, nothing else.
#include "sdp_transpose.h"

#include <algorithm>

namespace sdp {
namespace {

// 16-bit elements, 16-byte accesses on both sides.  Tile: 64 input rows x 64 columns.
// Requires C % 8 == 0, ld_in % 8 == 0, ld_out % 8 == 0, ld_out >= R and 16-byte aligned bases.  Output rows are written
// in whole 16-byte pieces: when R is no multiple of 8, elements R .. round_up(R, 8) - 1 of an output row become zeros.
// Up to kMaxTransposeJobs independent transposes run as one launch (grid.z = job), one tile a workgroup; workgroups beyond a
// job's own extent leave at once.  (The tiles in one linear order, as a carrying launch takes them: a division before the
// first load, 25.6 us instead of 24.1 for the four copies of T = 8192, d = 1536, p = 2048.)
__global__ __launch_bounds__(256) void transpose_rows_vec_kernel(TransposeJob j0, TransposeJob j1, TransposeJob j2, TransposeJob j3) {
    const int z = blockIdx.z;
    const TransposeJob jb = z == 0 ? j0 : z == 1 ? j1 : z == 2 ? j2 : j3;
    const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
    if (r0 >= jb.R || c0 >= jb.C) return;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kTransposeLds];
    TransposeTile tile;
    tile.index<false>(jb, r0, threadIdx.x);
    tile.load(jb, c0, threadIdx.x);
    tile.put(jb, r0, c0, lds, threadIdx.x);
    __syncthreads();
    TransposeTile::store(jb, r0, c0, lds, threadIdx.x);
}

// A copy of an fp32 operand whose memory an output of the same call takes over; no path that matters for speed.
__global__ __launch_bounds__(256) void copy_rows_f32_kernel(const float* in, const int32_t* rows, int C, int64_t n, float* out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = rows ? in[rows[i / C] * (int64_t)C + i % C] : in[i];
}

} // namespace

int copy_rows_f32(const float* in, const int32_t* rows, int R, int C, float* out, const char* name, hipStream_t s) {
    if (R < 1 || C < 1) return SDP_ERR_SHAPE;
    const int64_t n = (int64_t)R * C;
    ProfileScope ps(name, s);
    copy_rows_f32_kernel<<<(unsigned)std::min<int64_t>((n + 255) / 256, 4096), 256, 0, s>>>(in, rows, C, n, out);
    return launch_status();
}

static bool vec_ok(const TransposeJob& t) {
    return t.C % 8 == 0 && t.ld_out >= t.R && t.ld_in % 8 == 0 && t.ld_out % 8 == 0 && aligned16(t.in) && aligned16(t.out);
}

int transpose_rows(const void* in, int64_t ld_in, const int32_t* rows, int R, int C, void* out, int64_t ld_out,
                   const char* name, hipStream_t s) {
    const TransposeJob t{in, out, ld_in, ld_out, rows, R, C};
    return transpose_batch(&t, 1, name, s);
}

int side_jobs(const TransposeJob* t, int n, SideJobs* s) {
    *s = SideJobs{};
    if (n < 0 || n > kMaxTransposeJobs) return -1;
    int64_t tiles = 0;
    for (int i = 0; i < kMaxTransposeJobs; ++i) {
        if (i < n) {
            if (t[i].R < 1 || t[i].C < 1 || !vec_ok(t[i])) return -1;
            s->j[i] = t[i];
            tiles += ((int64_t)t[i].R + 63) / 64 * ((t[i].C + 63) / 64);
            if (tiles > 0x40000000) return -1;
        }
        s->end[i] = (int)tiles;
    }
    s->n = n;
    return (int)tiles;
}

int transpose_batch(const TransposeJob* t, int n, const char* name, hipStream_t s) {
    if (n < 1 || n > kMaxTransposeJobs) return SDP_ERR_INVALID_ARG;
    unsigned gx = 0, gy = 0;
    for (int i = 0; i < n; ++i) {
        if (t[i].R < 1 || t[i].C < 1) return SDP_ERR_SHAPE;
        if (!vec_ok(t[i])) return SDP_ERR_UNSUPPORTED;
        gx = std::max(gx, (unsigned)((t[i].R + 63) / 64));
        gy = std::max(gy, (unsigned)((t[i].C + 63) / 64));
    }
    if (gy > 65535) return SDP_ERR_SHAPE;
    TransposeJob j[kMaxTransposeJobs] = {};
    for (int i = 0; i < n; ++i) j[i] = t[i];
    ProfileScope ps(name, s);
    transpose_rows_vec_kernel<<<dim3(gx, gy, (unsigned)n), 256, 0, s>>>(j[0], j[1], j[2], j[3]);
    return launch_status();
}

} // namespace sdp
