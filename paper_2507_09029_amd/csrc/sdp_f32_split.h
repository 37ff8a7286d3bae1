// Part of sdp_gemm_f32.hip: fp32 contraction tiles on the bf16 matrix instructions.
//
// x 2^24 = h + m + l, each term the bf16 nearest to what the terms before it leave: 8 + 8 + 8 bits.  The scale makes this exact for every
// float below 2^103: the last bit of the smallest, 2^-149, becomes 2^-125, and no term is subnormal (without it operands below 2^-110
// lost bits, and those below 2^-134 all).  a b is then the sum of nine products, of which h h, h m, m h, m m, h l and l h are taken; the
// other three are below 2^-26 |a b|.  Six v_mfma_f32_32x32x16_bf16 (192 cycles) replace eight v_mfma_f32_32x32x2_f32 (512).  The five
// small products have an accumulator of their own, since a sum added to the large one is rounded at its size.  Error against 64 bits,
// normwise, one sum of N(0, 1) products, fp32 instruction / one accumulator / two: 32 terms 9.9e-8 / 3.7e-8 / 3.7e-8, 512 4.4e-7 /
// 3.5e-7 / 1.3e-7, 4096 1.1e-6 / 9.6e-7 / 3.7e-7; of terms in [1, 2], 512 3.4e-7 / 2.2e-7 / 1.1e-7.
// Operands that are not finite or of about 2^104 and more, and sums of 2^80 and more, leave no finite scaled output: a tile with such an
// output is computed again with the fp32 instruction.
//
// What bounds it: LDS.  A step of 32 depths of a 64 x 64 tile writes 24 KB of terms (64 bytes a cycle) and reads 48 KB of fragments (128),
// about 800 cycles, for 12 MFMAs of 32 cycles a SIMD; a step takes 0.46 - 0.52 us whether one, two or three workgroups share a CU.
// The vector instructions, 114 a wave and step, run between the MFMAs: beside MFMAs a SIMD issues one every 4 cycles, and a 16x16x32
// MFMA keeps it from that for 8 of its 16 cycles, a 32x32x16 one for 10 of its 32 (hence 32 x 32 fragments); v_dot2_f32_bf16, which
// would take a term's value off in one instruction instead of two, does not run beside an MFMA at all.  Tried: a third LDS stage,
// so that the next step's fragments are read between the MFMAs, 5 % slower (two workgroups a CU); 128 x 64 tiles 7 % faster from 4000
// tiles on and much slower below; terms split by each wave as it reads (tiles of 16 and 32), 10 % slower.
// Kernel times of both passes of a worker, fp32 instruction / split without the scale / so, us: T = 2048, d = 2048, p = 4000 2655 / 2150 / 2216;
// T = 1024, d = 1024, p = 2048 405 / 320 / 329; T = 1023, d = 511, p = 1535 324 / 224 / 228.
#pragma once

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4))); // four floats at any float's address

constexpr float kUp = 0x1p24f, kDown = 0x1p-48f; // an operand's scale, and what it takes a sum back
struct Terms {
    u32x4 h, m, l; // 8 bf16 each
};
// the terms of the floats 2 i and 2 i + 1 of eight
__device__ inline void split_pair(const f32x4 (&x)[2], int i, Terms& t) {
    auto pack = [](float p, float q) {
        uint32_t w = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)p, (__bf16)q});
        asm("" : "+v"(w)); // one value: the compiler would convert the lower half again where it is taken off
        return w;
    };
    const float a = kUp * x[i >> 1][2 * (i & 1)], b = kUp * x[i >> 1][2 * (i & 1) + 1];
    const uint32_t h = pack(a, b);
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xFFFF0000u);
    const uint32_t m = pack(ra, rb);
    t.h[i] = h, t.m[i] = m;
    t.l[i] = pack(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xFFFF0000u));
}

// One operand's step of 32 depths, R rows (M or N side), in LDS as three planes of bf16.  A thread moves PER pieces of 8 floats from
// memory through registers, where it splits them: each element is split once a workgroup.  Chunk c, c = 0 .. 3, stands for the
// depths 4 c .. 4 c + 3 and 16 + 4 c .. 16 + 4 c + 3, in both layouts; a fragment of half h is 32 rows of chunk 2 h + lane / 32.
//   rows        : plane [R rows][4 chunks of 16 bytes], chunk c of row r at c ^ turn(r): a 16-byte read serves lanes 0 .. 3, 12 .. 15
//                 and 20 .. 27 together (4 .. 11, 16 .. 19, 28 .. 31 next), 16 different places.  A thread's piece is a chunk, two loads
//                 of 16 bytes, each of which takes 64 contiguous bytes of 16 rows; a fragment is one 16-byte read.
//   depth-major : plane [32 depths][R / 16 granules of 16 rows]; a piece is 8 rows of one depth; a fragment is two transposing reads,
//                 4 depths x 16 rows for each 16 lanes.  Granule c of depth k sits at c ^ swap(k): the eight 32-byte pieces that
//                 32 lanes read then lie on distinct banks.
template <int R, bool DM, int THREADS>
struct SplitOperand {
    static constexpr int PLANE = R * 64, BYTES = 3 * PLANE, PER = R * 4 / THREADS;
    static constexpr int CPR = DM ? R / 8 : 4; // pieces per LDS row
    static_assert(R * 4 % THREADS == 0 && THREADS % CPR == 0 && (!DM || R == 64 || R == 128), "whole pieces");
    __device__ static int swap(int k) { return R == 64 ? k & 2 : 2 * (k & 3); }
    __device__ static int turn(int r) { return r >> 2 & 3; }
    __device__ static int line(int tid, int i) { return (tid + THREADS * i) / CPR; } // LDS row of piece i
    __device__ static int place(int tid, int i) {
        const int q = line(tid, i), c = tid % CPR;
        if constexpr (DM) return q * R * 2 + ((c >> 1 ^ swap(q)) * 32) + (c & 1) * 16;
        else return q * 64 + ((c ^ turn(q)) * 16);
    }
    __device__ static void stash(unsigned char* planes, const Terms& t, int i, int tid) { // piece i
        unsigned char* p = planes + place(tid, i);
        *(u32x4*)p = t.h, *(u32x4*)(p + PLANE) = t.m, *(u32x4*)(p + 2 * PLANE) = t.l;
    }
    // rows row0 .. row0 + 15 and those `apart` further of one plane (depth-major: apart = 16)
    __device__ static bf16x8 fragment(const unsigned char* plane, int row0, int apart, int h, int lane) {
        if constexpr (DM) {
            const int gi = lane >> 4, li = lane & 15;
            u32x2 w[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = 16 * e + 4 * (2 * h + (gi >> 1)) + (li >> 2);
                const unsigned char* p = plane + k * R * 2 + (((row0 >> 4) + (gi & 1) ^ swap(k)) * 32) + (li & 3) * 8;
                w[e] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p));
            }
            return __builtin_bit_cast(bf16x8, u32x4{w[0][0], w[0][1], w[1][0], w[1][1]});
        } else {
            const int l32 = lane & 31, r = row0 + (l32 & 15) + (l32 >> 4) * apart;
            return __builtin_bit_cast(bf16x8, *(const u32x4*)(plane + r * 64 + ((2 * h + (lane >> 5) ^ turn(r)) * 16)));
        }
    }
};

// Tile: BM x BN outputs (of both right operands: BN / 2 columns of each), KG teams of WM x WN waves.  Team g takes the depth steps (32) g,
// g + KG, ..., in two LDS stages of its own, with its next two steps in registers and one barrier a step:
//   step t : MFMAs on step t, between them step t + KG from registers, split, to the other stage; loads of step t + 3 KG
// The teams add up in LDS.  KG = 2 (one workgroup a CU) where the tiles do not fill the CUs twice: a SIMD needs two waves, since one
// alone issues a vector instruction every 5.5 cycles.
// Any strides and bases: loads of 16 bytes need no more than a float's alignment.  Depth K >= 32: the last step begins at K - 32 and
// takes as zeros, of the left operand, the depths that the step before had.  A depth-major operand's last tile begins BM (BN)
// before the extent's end and does not store what the tile before it does; rows beyond a row-major operand's are its last.
template <int KG, int EPI, bool ADM, bool BDM, bool AG>
struct SplitTile {
    static constexpr int BM = 64, BN = 64, WM = 2, WN = 2;
    static constexpr int TEAM = 64 * WM * WN, THREADS = KG * TEAM;
    static constexpr bool kTwoB = EPI == EPI_SWIGLU_FWD;
    static constexpr int COLS = kTwoB ? BN / 2 : BN; // of each right operand
    typedef SplitOperand<BM, ADM, TEAM> OA;
    typedef SplitOperand<BN, BDM, TEAM> OB;
    static constexpr int STAGE = OA::BYTES + OB::BYTES, LDS = KG * 2 * STAGE;
    // of the tile computed again: floats as they are
    typedef Operand<BM, 32, ADM> XA;
    typedef Operand<BN, 32, BDM> XB;
    static_assert((XA::FLOATS + XB::FLOATS) * 4 + 16 <= LDS && LDS <= 160 * 1024 && (!AG || ADM) && !(kTwoB && BDM), "fits");
    static_assert((KG == 1 || KG == 2) && BM == 32 * WM && BN == 32 * WN && THREADS * 32 + 16 <= LDS, "a fragment a wave; the teams' halves");

    __device__ static void run(const Dev& g, int block, unsigned char* smem) {
        const int team = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / TEAM);
        const int tid = threadIdx.x - team * TEAM, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int per = g.tiles_m * g.tiles_n;
        const int z = block / per, tile = block - z * per;
        const int m_lo = (tile % g.tiles_m) * BM, n_lo = (tile / g.tiles_m) * COLS;
        const int m0 = ADM && m_lo > g.M - BM ? g.M - BM : m_lo, n0 = BDM && n_lo > g.N - BN ? g.N - BN : n_lo;
        // the wave's part; of both right operands: 16 columns of each in a fragment, COLS apart in LDS
        const int pm = wave / WN * 32, pn = wave % WN * (kTwoB ? 16 : 32), apart = kTwoB ? COLS : 16;
        const float *gA = g.A, *gB = g.B;
        float* gC = g.C;
        if (g.nbatch > 0) {
            gA = z == 0 ? g.Ab[0] : (z == 1 ? g.Ab[1] : (z == 2 ? g.Ab[2] : g.Ab[3]));
            gB = z == 0 ? g.Bb[0] : (z == 1 ? g.Bb[1] : (z == 2 ? g.Bb[2] : g.Bb[3]));
            gC = z == 0 ? g.Cb[0] : (z == 1 ? g.Cb[1] : (z == 2 ? g.Cb[2] : g.Cb[3]));
        }

        // element offsets of this thread's pieces at depth 0, from the operand's base
        int64_t offa[OA::PER], offb[OB::PER];
        const float* baseb[OB::PER]; // kTwoB: of its right operand
        int cols[AG ? 8 : 1];        // AG: the piece's columns
#pragma unroll
        for (int i = 0; i < OA::PER; ++i) {
            const int q = OA::line(tid, i), c = tid % OA::CPR;
            if constexpr (ADM) {
                offa[i] = AG ? 0 : m0 + 8 * c;
            } else {
                int r = m0 + q;
                r = r < g.M ? r : g.M - 1;
                offa[i] = (int64_t)(g.ag ? g.ag[r] : r) * g.lda + 4 * c;
            }
        }
        if constexpr (AG) {
#pragma unroll
            for (int e = 0; e < 8; ++e) cols[e] = g.ag[m0 + 8 * (tid % OA::CPR) + e];
        }
#pragma unroll
        for (int i = 0; i < OB::PER; ++i) {
            const int q = OB::line(tid, i), c = tid % OB::CPR;
            if constexpr (BDM) {
                offb[i] = n0 + 8 * c;
            } else {
                int r = n0 + q % COLS;
                r = r < g.N ? r : g.N - 1;
                offb[i] = (int64_t)(g.bg ? g.bg[r] : r) * g.ldb + 4 * c;
            }
            if (kTwoB) baseb[i] = q < COLS ? g.B : g.B2;
        }

        const int n1 = (g.K + 31) / 32, n = EPI == EPI_DUAL_ACC ? 2 * n1 : n1;
        struct Raw {
            f32x4 a[OA::PER][2], b[OB::PER][2];
        };
        int listed[OB::PER]; // BDM: rows of the list for the next step to load
        auto first_of = [&](int t) { return 32 * (EPI == EPI_DUAL_ACC && t >= n1 ? t - n1 : t); }; // depth of step t, as it is counted
        auto depth = [&](int t) {                                                                 // and as it is read
            const int k0 = first_of(t);
            return k0 < g.K - 32 ? k0 : g.K - 32;
        };
        auto list = [&](int t) {
            if constexpr (BDM) {
                if (g.bg) {
                    const int32_t* q = g.bg + depth(t < n ? t : n - 1);
#pragma unroll
                    for (int i = 0; i < OB::PER; ++i) listed[i] = q[OB::line(tid, i)];
                }
            }
        };
        auto load = [&](int t, Raw& r) { // the list of step t has been asked for
            t = t < n ? t : n - 1;
            const bool second = EPI == EPI_DUAL_ACC && t >= n1;
            const int k = depth(t);
            const float *pa = second ? g.A2 : gA, *pb = second ? g.B2 : gB;
#pragma unroll
            for (int i = 0; i < OA::PER; ++i) {
                if constexpr (AG) {
                    const float* q = pa + (int64_t)(k + OA::line(tid, i)) * g.lda;
#pragma unroll
                    for (int e = 0; e < 8; ++e) r.a[i][e >> 2][e & 3] = q[cols[e]];
                } else {
                    const float* q = pa + offa[i] + (ADM ? (int64_t)(k + OA::line(tid, i)) * g.lda : k);
                    r.a[i][0] = *(const f32x4_any*)q;
                    r.a[i][1] = *(const f32x4_any*)(q + (ADM ? 4 : 16));
                }
            }
#pragma unroll
            for (int i = 0; i < OB::PER; ++i) {
                const float* q = (kTwoB ? baseb[i] : pb) + offb[i];
                if constexpr (BDM) q += (int64_t)(g.bg ? listed[i] : k + OB::line(tid, i)) * g.ldb;
                else q += k;
                r.b[i][0] = *(const f32x4_any*)q;
                r.b[i][1] = *(const f32x4_any*)(q + (BDM ? 4 : 16));
            }
        };
        // A step is partial where it reads depths that the step before has had: these count as zeros.  So do all depths of steps
        // beyond the last.
        auto partial = [&](int t) { return t >= n || (g.K % 32 != 0 && (t == n - 1 || (EPI == EPI_DUAL_ACC && t == n1 - 1))); };
        auto drop = [&](int t, f32x4& v, int k, bool along) {
            const int first = t < n ? first_of(t) - depth(t) : 32; // depths of the step that count: from here on
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + (along ? e : 0) < first) v[e] = 0.f;
        };
        auto drop_a = [&](int t, Raw& r) {
#pragma unroll
            for (int i = 0; i < OA::PER; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) drop(t, r.a[i][h], ADM ? OA::line(tid, i) : 4 * (tid % OA::CPR) + 16 * h, !ADM);
        };
        auto barrier = [&] {
            __builtin_amdgcn_sched_barrier(0);
            SDP_WAIT_LGKMCNT0();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };

        // the halves of a step have small-product accumulators of their own: an MFMA does not wait for the one before it
        f32x16 acc, low[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = low[0][e] = low[1][e] = 0.f;

        unsigned char* const stages = smem + team * 2 * STAGE;
        // Pair x of the next step's pieces; the last one of a piece sends it to LDS.
        constexpr int PAIRS = 4 * (OA::PER + OB::PER), MFMAS = 12;
        auto split = [&](unsigned char* st, const Raw& r, Terms& t, int x) {
            const int i = x / 4;
            split_pair(i < OA::PER ? r.a[i < OA::PER ? i : 0] : r.b[i < OA::PER ? 0 : i - OA::PER], x % 4, t);
            if (x % 4 == 3) {
                if (i < OA::PER) OA::stash(st, t, i, tid);
                else OB::stash(st + OA::BYTES, t, i - OA::PER, tid);
            }
        };
        // Everything runs unconditionally, which keeps a step one block of code: steps beyond the last are loads of the last one
        // again.  All fragments are asked for first.  drop_c: the step to split may be a partial one.
        auto step = [&](int t, unsigned char* st, unsigned char* into, Raw& next, auto drop_c) {
            if constexpr (decltype(drop_c)::value) {
                if (partial(t + KG)) drop_a(t + KG, next);
            }
            bf16x8 fa[3][2], fb[3][2];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    fa[p][h] = OA::fragment(st + p * OA::PLANE, pm, 16, h, lane);
                    fb[p][h] = OB::fragment(st + OA::BYTES + p * OB::PLANE, pn, apart, h, lane);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr int TA[6] = {0, 0, 1, 1, 0, 2}, TB[6] = {0, 1, 0, 1, 2, 0}; // h h, h m, m h, m m, h l, l h
            Terms terms;
#pragma unroll
            for (int m = 0; m < MFMAS; ++m) {
                // h h of the first half, the small products of both in turn, h h of the second half
                const int q = m == 0 || m == MFMAS - 1 ? 0 : (m + 1) / 2, h = m == 0 ? 0 : m == MFMAS - 1 ? 1 : (m + 1) % 2;
                f32x16& c = q == 0 ? acc : low[h]; // B first: a lane then holds 4 consecutive columns of one row
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[TB[q]][h], fa[TA[q]][h], c, 0, 0, 0);
                // two pairs at a time, whose instructions fill each other's wait states
                constexpr int P2 = PAIRS / 2;
                if (m * P2 / MFMAS != (m + 1) * P2 / MFMAS) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int x = m * P2 / MFMAS; x < (m + 1) * P2 / MFMAS; ++x) {
                        split(into, next, terms, 2 * x);
                        split(into, next, terms, 2 * x + 1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            load(t + 3 * KG, next);
            list(t + 4 * KG);
            barrier();
        };
        Raw ra, rb;
        list(team);
        load(team, ra);
        list(team + KG);
        load(team + KG, rb);
        list(team + 2 * KG);
        if (partial(team)) drop_a(team, ra);
        {
            Terms terms;
#pragma unroll
            for (int x = 0; x < PAIRS; ++x) split(stages, ra, terms, x);
        }
        load(team + 2 * KG, ra);
        list(team + 3 * KG);
        barrier();
        const int rounds = (n + KG - 1) / KG, whole = (n1 - 1) / KG; // of all teams; steps below KG whole are whole ones
        int u = 0;
        for (; u + 3 <= whole; u += 2) { // splits the steps of rounds u + 1, u + 2
            step(team + KG * u, stages, stages + STAGE, rb, std::false_type{});
            step(team + KG * (u + 1), stages + STAGE, stages, ra, std::false_type{});
        }
        for (; u < rounds; u += 2) {
            step(team + KG * u, stages, stages + STAGE, rb, std::true_type{});
            if (u + 1 < rounds) step(team + KG * (u + 1), stages + STAGE, stages, ra, std::true_type{});
        }

        // G and U of the whole fragment are asked for at once: read where they are used, each waits behind the stores of the one before
        // it, which the compiler may not move it across (6.5 -> 4.7 us a round of tiles: T = 1692, d = 828, n = 5028 175.6 -> 163.9 us,
        // T = 1592, d = 524, n = 2884 76.2 -> 71.1)
        f32x4 gu[4][2];
        if constexpr (EPI == EPI_SWIGLU_BWD) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (KG == 1 || q % 2 == team) {
                    gu[q][0] = row_of_four(g, g.Gin, g.ldg, m0 + pm + l32, n0 + pn + 8 * q + 4 * lhi);
                    gu[q][1] = row_of_four(g, g.Uin, g.ldg, m0 + pm + l32, n0 + pn + 8 * q + 4 * lhi);
                }
        }
        acc = (acc + (low[0] + low[1])) * kDown;
        // element 4 q + r of acc: row l32 of A's fragment, row 8 q + 4 lhi + r of B's.  KG = 2: team 0 finishes q = 0 and 2, team 1
        // the others; each leaves the other's in LDS.
        auto part = [&](int q) { return f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]}; };
        auto mine = [&](int q) { return KG == 1 || q % 2 == team; };
        int* const again = (int*)(smem + LDS - 16);
        if (threadIdx.x == 0) *again = 0;
        if constexpr (KG == 2) {
            float* const put = (float*)smem + ((team ^ 1) * TEAM + tid) * 8;
            const float* const get = (const float*)smem + threadIdx.x * 8;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (!mine(q)) *(f32x4*)(put + 4 * (q / 2)) = part(q);
            barrier();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (mine(q)) {
                    const f32x4 v = *(const f32x4*)(get + 4 * (q / 2));
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[4 * q + e] += v[e];
                }
        }
        float bad = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) bad += acc[e] * 0.f;
        barrier();
        if (bad != 0.f) *again = 1;
        barrier();
        if (*again) { // every team the whole tile
            float* const fl = (float*)smem;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.f;
            barrier();
            for (int t = 0; t < n; ++t) {
                list(t);
                load(t, ra);
                if (partial(t)) {
                    drop_a(t, ra);
#pragma unroll
                    for (int i = 0; i < OB::PER; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h) drop(t, ra.b[i][h], BDM ? OB::line(tid, i) : 4 * (tid % OB::CPR) + 16 * h, !BDM);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int i = 0; i < OA::PER; ++i)
                        *(f32x4*)(fl + OA::line(tid, i) * XA::LD + (ADM ? 8 * (tid % OA::CPR) + 4 * h : 4 * (tid % OA::CPR) + 16 * h)) = ra.a[i][h];
#pragma unroll
                    for (int i = 0; i < OB::PER; ++i)
                        *(f32x4*)(fl + XA::FLOATS + OB::line(tid, i) * XB::LD + (BDM ? 8 * (tid % OB::CPR) + 4 * h : 4 * (tid % OB::CPR) + 16 * h)) =
                            ra.b[i][h];
                }
                barrier();
                for (int k = lhi; k < 32; k += 2) {
                    const int r = pn + (l32 & 15) + (l32 >> 4) * apart;
                    const float fa = fl[ADM ? k * XA::LD + pm + l32 : (pm + l32) * XA::LD + k];
                    const float fb = fl[XA::FLOATS + (BDM ? k * XB::LD + r : r * XB::LD + k)];
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb, fa, acc, 0, 0, 0);
                }
                barrier();
            }
        }
        const int m = m0 + pm + l32;
        if (ADM && m < m_lo) return;
#pragma unroll
        for (int q = 0; q < (kTwoB ? 2 : 4); ++q)
            if (mine(q))
                emit<EPI, BDM>(g, gC, m, n0 + pn + 8 * q + 4 * lhi, part(q), part(kTwoB ? q + 2 : q), n_lo, EPI == EPI_SWIGLU_BWD ? gu[q] : nullptr);
    }
};

template <int KG, int EPI, bool ADM, bool BDM, bool AG>
__global__ __launch_bounds__(256 * KG, 2) void gemm_f32_split_kernel(Dev g) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[SplitTile<KG, EPI, ADM, BDM, AG>::LDS];
    SplitTile<KG, EPI, ADM, BDM, AG>::run(g, blockIdx.x, lds);
}

template <int KG, int EPI, bool ADM, bool BDM, bool AG>
int launch_split(Dev g, const char* name, hipStream_t s) {
    constexpr int COLS = SplitTile<KG, EPI, ADM, BDM, AG>::COLS;
    g.tiles_m = (g.M + 63) / 64, g.tiles_n = (g.N + COLS - 1) / COLS;
    const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * (g.nbatch > 0 ? g.nbatch : 1); // below 2^23 (split_pays)
    profile_shape(name, 64, COLS, 0, KG == 1 ? F32_SPLIT : F32_SPLIT_TEAMS);
    ProfileScope ps(name, s);
    gemm_f32_split_kernel<KG, EPI, ADM, BDM, AG><<<(unsigned)blocks, 256 * KG, 0, s>>>(g);
    return launch_status();
}
