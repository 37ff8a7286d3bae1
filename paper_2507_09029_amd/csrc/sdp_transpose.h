// Device side of the (gathered) transposes of 16-bit matrices: 64 x 64 element tiles through LDS, 256 threads a tile,
// 16-byte accesses on both sides.  out[c][r] = in[rows ? rows[r] : r][c]; see transpose_rows for what a job requires.
// Used by the launches of their own (sdp_transpose.hip) and by launches of other kernels that carry transposes which a
// later kernel needs as extra workgroups.
#pragma once
#include "sdp_internal.h"

namespace sdp {

constexpr int kTransposeRow = 64 * 2 + 16;         // LDS bytes of a tile row
constexpr int kTransposeLds = 64 * kTransposeRow;  // and of a tile

// j[0], j[1], j[2] or j[3], the first whose condition holds.  Field by field: a runtime index into a kernel argument, or a
// reference selected among its elements, goes through scratch.
__device__ inline TransposeJob pick_job(const TransposeJob (&j)[kMaxTransposeJobs], bool z0, bool z1, bool z2) {
    static_assert(kMaxTransposeJobs == 4, "one condition per job but the last");
    return {z0 ? j[0].in : z1 ? j[1].in : z2 ? j[2].in : j[3].in,
            z0 ? j[0].out : z1 ? j[1].out : z2 ? j[2].out : j[3].out,
            z0 ? j[0].ld_in : z1 ? j[1].ld_in : z2 ? j[2].ld_in : j[3].ld_in,
            z0 ? j[0].ld_out : z1 ? j[1].ld_out : z2 ? j[2].ld_out : j[3].ld_out,
            z0 ? j[0].rows : z1 ? j[1].rows : z2 ? j[2].rows : j[3].rows,
            z0 ? j[0].R : z1 ? j[1].R : z2 ? j[2].R : j[3].R,
            z0 ? j[0].C : z1 ? j[1].C : z2 ? j[2].C : j[3].C,
            {z0 ? j[0].heads.width : z1 ? j[1].heads.width : z2 ? j[2].heads.width : j[3].heads.width,
             z0 ? j[0].heads.magic : z1 ? j[1].heads.magic : z2 ? j[2].heads.magic : j[3].heads.magic,
             z0 ? j[0].heads.held : z1 ? j[1].heads.held : z2 ? j[2].heads.held : j[3].heads.held,
             z0 ? j[0].heads.all : z1 ? j[1].heads.all : z2 ? j[2].heads.all : j[3].heads.all}};
}

// Tile at input rows r0 .., columns c0 .. of a job.  Thread t moves rows t / 8 and t / 8 + 32, columns 8 (t % 8) ..  The
// loads are unconditional (rows and columns clamped, what lies outside becomes zeros on the way to LDS), so that those of
// several tiles can be in flight together.
struct TransposeTile {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
    int row[2];
    u32x4 v[2];
    // HEADS: the rows may be a list of heads (the attention's; the look-up makes the MLP's carried transposes 2.4 us longer)
    template <bool HEADS>
    __device__ void index(const TransposeJob& jb, int r0, int t) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = r0 + (t >> 3) + 32 * h, rc = r < jb.R ? r : jb.R - 1;
            row[h] = HEADS ? listed_row(jb.rows, jb.heads, rc) : jb.rows ? jb.rows[rc] : rc;
        }
    }
    __device__ void load(const TransposeJob& jb, int c0, int t) {
        const int c = c0 + (t & 7) * 8;
#pragma unroll
        for (int h = 0; h < 2; ++h) v[h] = *(const u32x4*)((const uint16_t*)jb.in + (int64_t)row[h] * jb.ld_in + (c < jb.C ? c : 0));
    }
    __device__ void put(const TransposeJob& jb, int r0, int c0, unsigned char* tile, int t) const {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = (t >> 3) + 32 * h;
            const bool in = r0 + r < jb.R && c0 + (t & 7) * 8 < jb.C;
            *(u32x4*)(tile + r * kTransposeRow + (t & 7) * 16) = in ? v[h] : u32x4{0u, 0u, 0u, 0u};
        }
    }
    // A transposing read hands lane n of 16, as its e-th element, position n % 4 of the 8 bytes that lane 4 e + n / 4
    // addressed.  Two of them give a lane 8 consecutive input rows of one column, one 16-byte piece of an output row; the
    // 64 lanes cover the 8 pieces of 8 output rows.
    __device__ static void store(const TransposeJob& jb, int r0, int c0, const unsigned char* tile, int t) {
        const int lane = t & 63, gi = lane >> 4, li = lane & 15;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c4 = 8 * (2 * (t >> 6) + h) + 4 * (gi & 1), strip = 32 * (gi >> 1);
            const unsigned char* p = tile + (strip + 8 * (li & 3) + (li >> 2)) * kTransposeRow + c4 * 2;
            const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p));
            const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * kTransposeRow)));
            const int c = c0 + c4 + (li & 3), r = r0 + strip + 8 * (li >> 2);
            if (c < jb.C && r < jb.R) *(u32x4*)((uint16_t*)jb.out + (int64_t)c * jb.ld_out + r) = u32x4{a[0], a[1], b[0], b[1]};
        }
    }
};

// Transposes that ride on another kernel's launch: their tiles in one linear order, job after job.
struct SideJobs {
    TransposeJob j[kMaxTransposeJobs];
    int end[kMaxTransposeJobs]; // tiles of the jobs up to and including this one
    int n;                      // jobs; 0 = none
};

// N tiles at once by 256 threads (t = 0 .. 255), tiles N w .. N w + N - 1 (the last tile again beyond it); lds: N x
// kTransposeLds bytes of these threads' own.  Every thread of the workgroup has to get here (barrier).
template <int N, bool HEADS = false>
__device__ inline void side_transposes(const SideJobs& s, int w, unsigned char* lds, int t) {
    TransposeTile tile[N];
    TransposeJob jb[N];
    int r0[N], c0[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        int id = N * w + i;
        id = id < s.end[3] ? id : s.end[3] - 1;
        const bool z0 = id < s.end[0], z1 = id < s.end[1], z2 = id < s.end[2];
        jb[i] = pick_job(s.j, z0, z1, z2);
        const int first = z0 ? 0 : z1 ? s.end[0] : z2 ? s.end[1] : s.end[2];
        const int tr = (jb[i].R + 63) / 64;
        r0[i] = (id - first) % tr * 64, c0[i] = (id - first) / tr * 64;
        tile[i].template index<HEADS>(jb[i], r0[i], t);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) tile[i].load(jb[i], c0[i], t);
#pragma unroll
    for (int i = 0; i < N; ++i) tile[i].put(jb[i], r0[i], c0[i], lds + i * kTransposeLds, t);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) TransposeTile::store(jb[i], r0[i], c0[i], lds + i * kTransposeLds, t);
}

} // namespace sdp
