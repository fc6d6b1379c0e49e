// Complex64 GEMM on CDNA4 FP32 matrix cores: the dense products of the method (ADMM solver section:
// r = D X - U in the objective of eq. X2LQR_lst, W = D^H r in the gradient equations DXLR, the line-search
// products a = D X1 and b = D X2) and the stages of the tile forms.
//
// Every wave owns one 32 x 32 block of C (GM_LINE: the same block of a and b) and feeds its MFMAs from
// global memory through registers, without LDS and without a barrier in the k loop. An FP32 MFMA takes 64
// cycles, so the 8 KiB of operands that a wave needs per 16 complex k (1536 cycles of products in the
// three-product form) come to 21 bytes per cycle and CU, a third of what L1 delivers; the other waves of the
// SIMD (3 to 4, 2 or 3 in GM_LINE) cover the loads, and in small launches the products of the chunk before
// (AHEAD). The matrix core rate is what bounds it. Measured, TFLOP/s counted 8mnk with
// the 128 x 128 tiles staged through LDS that this replaces in brackets: one problem of 1024^2, three
// products: r = D X - U 58 us (252), D^H r 56 (223), [a | b] 107 (234); one of 4096 x 2048: 1500 us (1678),
// 1432 (1547), 2834 (3077); 34 of 1024^2, four-product form 144 (144), three-product form 136 (125).
//   KS = 1: a workgroup is 4 waves (2 x 2) on a 64 x 64 tile, which share its operands through L1.
//   KS = 4: a workgroup's 4 waves share one 32 x 32 block and each takes every fourth chunk of k; their
//     sums are added in LDS in a fixed order. Four times as many waves, each a quarter as long, for
//     problems that would leave SIMDs idle or a last round nearly empty. The order of the sums is
//     another one, so a problem's own sizes choose the form (gemm_split_k), not its batch.
//
// 4M (four products): Re C += Ar Br, Im C += Ar Bi, Re C += (-Ai) Bi, Im C += Ai Br: 8MNK flops.
// 3M (three products): T1 = Ar Br, T2 = Ai Bi, T3 = (Ar + Ai)(Br + Bi), Re C = T1 - T2, Im C = T3 - T1 - T2:
//   6MNK flops, at the price of one extra rounding level in Im C (the sums and the final differences).
// One v_mfma_f32_32x32x2_f32 multiplies two complex k of one of these products; a lane ends with whole
// complex entries of one column.
//
// Epilogues: GM_STORE (C = AB), GM_RESID (C = AB - U plus FP64 partial sums of |C|^2) and GM_LINE (a and b
// plus FP64 partial sums of Re<r,a>, |a|^2, Re<r,b>, Re<a,b>, |b|^2 for the exact line search). GM_LINE unsplit, three
// products, has two registers too few for three waves per SIMD in its epilogue: they go through scratch once a wave,
// outside the k loop.
//
// Operands are padded to whole 64-tiles with zeros, or read where the caller has them: no load carries a bounds
// check (they are buffer loads: anything past an operand's last row reads zero), and what a row-major operand
// holds past its last column only reaches columns or rows of C that are not stored (Mc x Nc), not summed
// (Me x Ne) or never read. Blocks outside the true sizes (Mt x Nt) are written as zeros without their products.
#include <algorithm>
#include <type_traits>

#include "extents.hpp"
#include "gemm_common.hpp"

namespace tlr {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

namespace {

__device__ __forceinline__ float flip(float v, uint32_t sign) { return __uint_as_float(__float_as_uint(v) ^ sign); }

// The operands of one chunk of CH complex k as loaded. Every step multiplies two k, one per lane half h. A
// row-major A comes in 16-byte loads, k = 4 q + 2 h and the next one: step (q, e) then multiplies 4 q + e and
// 4 q + e + 2. The tile stages multiply k and k + 1 instead, for which the lane halves exchange one entry of
// each load: their products are carried from iteration to iteration, and at 2 Hz 100 iterations amplify any
// rounding past what FP32 state allows (5.6e-5 in X; this order ends at 3.7e-5, the other at 7.3e-5, at 6 %
// less time per stage).
template <bool TA, int HB, int NB, int CH>
struct Chunk {
    float4 a4[HB][TA ? 1 : CH / 4];
    float2 a2[HB][TA ? CH / 2 : 1];
    float2 b[NB][CH / 2];
};

constexpr int SCHED_ALU = 0x6;   // only ALU instructions may be moved across the barrier

// AHEAD: a chunk's loads stay in flight during the products of the one before. Without it they do not: a branch
// around the next chunk's loads makes the wait for the chunk at hand a wait for all, and the other waves cover that.
template <int MODE, bool M3, int ROLE, int KS, bool BIG, bool AHEAD>
__global__ __launch_bounds__(256, BIG ? 2 : 3) void cgemm_kernel(GemmArgs g) {
    constexpr bool TA = ROLE == GR_TILE_TA_CB || ROLE == GR_ADJOINT;
    constexpr bool STAGE = ROLE == GR_TILE || ROLE == GR_TILE_TA_CB;
    constexpr int HK = STAGE ? 1 : 2;              // k between the lane halves of a step
    constexpr int HB = BIG ? 2 : 1;                // row blocks of a wave
    constexpr int NB = (MODE == GM_LINE || BIG) ? 2 : 1;   // column blocks (GM_LINE: of X1 and of X2)
    constexpr int CB = MODE == GM_LINE ? 1 : NB;   // blocks of 32 columns of C
    constexpr int NT = M3 ? 3 : 2;                 // accumulators per block: T1, T2, T3 or Re, Im
    constexpr int WV = KS == 1 ? 2 : 1;            // waves per workgroup tile row and column
    // complex k per chunk (one round of loads). GM_LINE takes 8: its accumulators and two column blocks then
    // fit three waves per SIMD instead of two (64 problems of 512^2, split: 892 us, with 16: 957)
    constexpr int CH = BIG && M3 ? 4 : NB == 2 ? 8 : 16;
    // k that a wave of a split contraction takes at a time, in chunks: the same for every tile, as the order of the sums
    constexpr int UNIT = KS == 1 ? CH : MODE == GM_LINE ? 8 : 16;
    constexpr int SUB = UNIT / CH;

    // workgroup -> batch entry and tile. Consecutive workgroups go to the eight XCDs in turn. Dense products:
    // contiguous tile ranges of an entry per XCD; tile stages, whose entries are small: whole entries per XCD,
    // so that its L2 fetches their operands once (32 frequencies of 4096 x 2048: gradient stages 3 % faster).
    // Either way tiles are grouped by 8 tile rows, which read few rows of A and few columns of B.
    const int nwg = gridDim.x;
    int zz = blockIdx.y, pid = blockIdx.x;
    if (STAGE && zz < (int)(gridDim.y & ~7u)) {
        const int lin = zz * nwg + pid;
        zz = ((lin >> 3) / nwg) * 8 + (lin & 7);
        pid = (lin >> 3) % nwg;
    } else if ((nwg & 7) == 0) {
        pid = (pid & 7) * (nwg >> 3) + (pid >> 3);
    }
    const int z = g.nz2 > 1 ? zz / g.nz2 : zz;
    int z2 = g.nz2 > 1 ? zz % g.nz2 : 0;
    int z3 = 0, z4 = 0;
    if (MODE == GM_STORE && STAGE) {
        if (g.nz4 > 1) {
            z4 = z2 % g.nz4;
            z2 = z2 / g.nz4;
        }
        if (g.nz3 > 1) {
            z3 = z2 % g.nz3;
            z2 = z2 / g.nz3;
        }
    }
    const float2 *A = g.A + z * g.sA + z2 * g.sA2 + z3 * g.sA3 + z4 * g.sA4;
    const float2 *B = g.B + z * g.sB + z2 * g.sB2 + z3 * g.sB3 + z4 * g.sB4;

    const int per_group = 8 * g.tiles_n;
    const int grp = pid / per_group;
    const int gsz = min(g.tiles_m - 8 * grp, 8);
    const int tm = 8 * grp + (pid % per_group) % gsz;
    const int tn = (pid % per_group) / gsz;

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int j32 = lane & 31, half = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = 32 * HB * (tm * WV + (KS == 1 ? wm : 0));   // the wave's first row and column
    const int n0 = 32 * CB * (tn * WV + (KS == 1 ? wn : 0));

    const __amdgpu_buffer_rsrc_t rsA =
        __builtin_amdgcn_make_buffer_rsrc(scalar(A), (short)0, (int)g.bytesA, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB =
        __builtin_amdgcn_make_buffer_rsrc(scalar(B), (short)0, (int)g.bytesB, 0x00020000);
    uint32_t offA[HB];
    offA[0] = TA ? (uint32_t)(((int64_t)HK * half * g.lda + m0 + j32) * 8)
                 : (uint32_t)(((int64_t)(m0 + j32) * g.lda + 2 * half) * 8);
    if (HB == 2) offA[HB - 1] = offA[0] + (uint32_t)(TA ? 32 * 8 : 32 * g.lda * 8);
    uint32_t offB[NB];
    offB[0] = (uint32_t)(((int64_t)HK * half * g.ldb + n0 + j32) * 8);
    if (NB == 2) offB[NB - 1] = offB[0] + (uint32_t)((MODE == GM_LINE ? g.b2_off : 32) * 8);

    auto k_of = [](int s) { return HK == 2 ? 4 * (s >> 1) + (s & 1) : 2 * s; };   // of lane half 0 in step s
    auto load = [&](Chunk<TA, HB, NB, CH> &c, int k0, bool b2) {
#pragma unroll
        for (int h = 0; h < HB; ++h) {
            if constexpr (TA) {
#pragma unroll
                for (int s = 0; s < CH / 2; ++s) {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rsA, (int)offA[h], (int)((uint32_t)(k0 + k_of(s)) * (uint32_t)g.lda * 8u), 0);
                    c.a2[h][s] = make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
                }
            } else {
#pragma unroll
                for (int q = 0; q < CH / 4; ++q) {
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsA, (int)(offA[h] + 32 * q), k0 * 8, 0);
                    c.a4[h][q] = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
                }
            }
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            if (n == 1 && !b2) continue;
#pragma unroll
            for (int s = 0; s < CH / 2; ++s) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rsB, (int)offB[n], (int)((uint32_t)(k0 + k_of(s)) * (uint32_t)g.ldb * 8u), 0);
                c.b[n][s] = make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
            }
        }
    };

    floatx16 acc[HB][NB][NT];
#pragma unroll
    for (int h = 0; h < HB; ++h)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int p = 0; p < NT; ++p)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[h][n][p][r] = 0.f;

    constexpr uint32_t conj_a = ROLE == GR_ADJOINT ? 0x80000000u : 0u;
    constexpr uint32_t conj_b = ROLE == GR_TILE_TA_CB ? 0x80000000u : 0u;
    auto mfma = [](float a, float b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); };
    auto compute = [&](const Chunk<TA, HB, NB, CH> &c, auto nb_tag) {
        constexpr int NBC = decltype(nb_tag)::value;   // column blocks with products in this chunk
#pragma unroll
        for (int s = 0; s < CH / 2; ++s) {
            float ar[HB], ai[HB];
#pragma unroll
            for (int h = 0; h < HB; ++h) {
                if constexpr (TA) {
                    ar[h] = c.a2[h][s].x;
                    ai[h] = flip(c.a2[h][s].y, conj_a);
                } else {
                    const float4 v = c.a4[h][s >> 1];
                    if constexpr (STAGE) {   // (k, k + 1 | k + 2, k + 3) -> (k | k + 1) and (k + 2 | k + 3)
                        const u32x2 re = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.x), __float_as_uint(v.z), false, false);
                        const u32x2 im = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.y), __float_as_uint(v.w), false, false);
                        ar[h] = __uint_as_float((s & 1) ? re.y : re.x);
                        ai[h] = __uint_as_float((s & 1) ? im.y : im.x);
                    } else {
                        ar[h] = (s & 1) ? v.z : v.x;
                        ai[h] = (s & 1) ? v.w : v.y;
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < (M3 ? 3 : 4); ++p)
#pragma unroll
                for (int h = 0; h < HB; ++h)
#pragma unroll
                    for (int n = 0; n < NBC; ++n) {
                        const float br = c.b[n][s].x, bi = flip(c.b[n][s].y, conj_b);
                        floatx16 *d = acc[h][n];
                        if constexpr (M3) d[p] = p == 0 ? mfma(ar[h], br, d[p]) : p == 1 ? mfma(ai[h], bi, d[p]) : mfma(ar[h] + ai[h], br + bi, d[p]);
                        else if (p & 1) d[1] = p == 1 ? mfma(ar[h], bi, d[1]) : mfma(ai[h], br, d[1]);
                        else d[0] = p == 0 ? mfma(ar[h], br, d[0]) : mfma(-ai[h], bi, d[0]);
                    }
        }
    };

    // the chunks of this wave: every KS-th unit's; GM_LINE tile stages: b over the first K2 k only
    constexpr bool SPLIT_K2 = MODE == GM_LINE && STAGE;
    const bool inside = m0 < g.Mt && n0 < g.Nt;
    const int own = KS == 1 ? 0 : wave;
    const int nc = inside ? (g.K / UNIT - own + KS - 1) / KS * SUB : 0;
    const int nc2 = (SPLIT_K2 && g.K2 > 0) ? g.K2 / CH : nc;
    auto k_at = [&](int c) { return KS == 1 ? c * CH : (c / SUB * KS + own) * UNIT + c % SUB * CH; };
    auto chunks = [&](int c, int end, auto nb_tag) {
        Chunk<TA, HB, NB, CH> r0, r1;
        constexpr bool B2 = decltype(nb_tag)::value > 1;
        if (c < end) load(r0, k_at(c), B2);
        if constexpr (AHEAD) {
            for (; c + 1 < end; c += 2) {
                load(r1, k_at(c + 1), B2);
                __builtin_amdgcn_sched_barrier(SCHED_ALU);
                compute(r0, nb_tag);
                load(r0, k_at(min(c + 2, end - 1)), B2);
                __builtin_amdgcn_sched_barrier(SCHED_ALU);
                compute(r1, nb_tag);
            }
            if (c < end) compute(r0, nb_tag);
        } else {
            for (; c < end; c += 2) {
                if (c + 1 < end) load(r1, k_at(c + 1), B2);
                compute(r0, nb_tag);
                if (c + 1 < end) {
                    if (c + 2 < end) load(r0, k_at(c + 2), B2);
                    compute(r1, nb_tag);
                }
            }
        }
    };
    chunks(0, nc2, std::integral_constant<int, NB>{});
    if constexpr (SPLIT_K2) chunks(nc2, nc, std::integral_constant<int, 1>{});

    EpiArgs ea;
    ea.C = g.C + z * g.sC + z2 * g.sC2 + z3 * g.sC3 + z4 * g.sC4;
    ea.C2 = MODE == GM_LINE ? g.C2 + z * g.sC + z2 * g.sC2 : nullptr;
    ea.ldc = g.ldc;
    ea.E = MODE == GM_STORE ? nullptr : g.E + z * g.sE + z2 * g.sE2;
    ea.lde = g.lde;
    ea.Me = g.Me;
    ea.Ne = g.Ne;
    ea.Mc = g.Mc;
    ea.Nc = g.Nc;
    ea.partials = MODE == GM_STORE ? nullptr : g.partials + z * g.sP + z2 * g.sP2;
    ea.nblk = g.N >> 5;
    ea.scat_kp = g.scat_kp;
    ea.scat_w = g.scat_w;
    ea.scat_lim = g.scat_lim;
    ea.scat_js = g.scat_js;
    constexpr int COLS = MODE != GM_STORE ? COL_PLAIN : STAGE ? COL_SCAT : ROLE == GR_DENSE ? COL_MAP : COL_PLAIN;
    ea.cmap = COLS == COL_MAP ? g.cmap + z * g.s_cmap : nullptr;
    block_epilogue<MODE, COLS, KS, HB, CB>(
        ea,
        [&](int h, int n, int r) {
            const floatx16 *d = acc[h][n];
            if constexpr (M3) return make_float2(d[0][r] - d[1][r], d[NT - 1][r] - d[0][r] - d[1][r]);
            else return make_float2(d[0][r], d[1][r]);
        },
        m0, n0);
}

// Three products in full launches do better without AHEAD (the results are the same): their SIMDs are full, and a
// sum of the operands per product lets the scheduler fill the waits. us, without and with it:
//   r = D X - U, D^H r, [a | b] of 448^2 15, 14, 23 and 14, 13, 21; of 1024^2 (1024 workgroups) 64, 62, 118 and 65, 62,
//   135; 16 of 1024^2 806, 785, 1550 and 828, 794, 1557; the line stages of one problem of tiles 128 (256 to 1024
//   workgroups) 102 and 95, of 8 problems 580 and 590.
// Four products and the 2 x 2 wave tiles always take it: 448^2 15, 14, 23 us without, 14, 14, 21 with it; D^H r of
// 4096 x 2048 1482 and 1436.
constexpr int64_t AHEAD_MAX_WG = 1023;
template <int MODE, bool M3, int ROLE, int KS, bool BIG = false>
hipError_t go(const GemmArgs &a, int batch, hipStream_t s) {
    const dim3 grid(a.tiles_m * a.tiles_n, batch);
    if constexpr (M3 && !BIG) {
        if ((int64_t)grid.x * batch > AHEAD_MAX_WG) {
            hipLaunchKernelGGL((cgemm_kernel<MODE, M3, ROLE, KS, BIG, false>), grid, dim3(256), 0, s, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((cgemm_kernel<MODE, M3, ROLE, KS, BIG, true>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

// Wave tiles of 2 x 2 blocks, in GM_LINE of two row blocks of a and of b: half the operand traffic per product, for two
// waves per SIMD instead of three or four. They pay where the workgroups fill the chip (KS = 1: two per CU; a split
// block's are shorter: four times) and the k loop is long against prologue and epilogue. The results are the same. us without and with them, three products:
//   GM_STORE: D^H r of 8 problems of 4096 x 2048 12.2 and 11.6 ms, of one 1.508 and 1.455; the gradient
//     stages of 8 problems of 1024^2, tiles 128, rank 16 (512 workgroups, K = 128 and 256) 184 and 171 us, stage 1 of the
//     line products with rank 24 (K = 128) 13 of 550 us less; split, 16 problems of 1024^2 789 and 748, 64 of 512^2 437 and 410.
//   GM_RESID, split only: 812 and 773, 468 and 437. (A wave alone has too few registers for its epilogue: 1490 and 1488
//     for 4096 x 2048, four products 996 and 1020 for 16 problems of 1024^2.)
//   GM_LINE: 4096 x 2048 2930 and 2834; split 1560 and 1505, 875 and 825, one problem of 1600^2 (1250 workgroups) 407
//     and 429. Tile stages 940 and 930 at most, four products within 1 %.
constexpr int64_t BIG_MIN_WG = 512, BIG_MIN_WG_SPLIT = 2048;
constexpr int BIG_MIN_K = 128;
template <int MODE, bool M3, int ROLE, int KS>
hipError_t go_big(GemmArgs a, int batch, hipStream_t s) {
    constexpr int WT = KS == 1 ? 64 : 32;   // the launcher's tiles
    constexpr bool DENSE3 = M3 && (ROLE == GR_DENSE || ROLE == GR_ADJOINT);
    if constexpr (MODE == GM_STORE ? KS == 1 || DENSE3 : DENSE3 && (MODE == GM_LINE || KS > 1)) {
        const bool wide = MODE != GM_LINE;   // two blocks of columns too; GM_LINE has a's and b's
        if (a.M % (2 * WT) == 0 && a.N % (wide ? 2 * WT : WT) == 0 && a.K >= BIG_MIN_K &&
            (int64_t)(a.tiles_m / 2) * (wide ? a.tiles_n / 2 : a.tiles_n) * batch >=
                (KS == 1 ? BIG_MIN_WG : BIG_MIN_WG_SPLIT)) {
            a.tiles_m /= 2;
            if (wide) a.tiles_n /= 2;
            return go<MODE, M3, ROLE, KS, true>(a, batch, s);
        }
    }
    return go<MODE, M3, ROLE, KS>(a, batch, s);
}

template <bool M3>
hipError_t go_dense(int mode, const GemmArgs &a, int batch, hipStream_t s, int role, bool split) {
    if (role == GR_ADJOINT)
        return split ? go_big<GM_STORE, M3, GR_ADJOINT, 4>(a, batch, s) : go_big<GM_STORE, M3, GR_ADJOINT, 1>(a, batch, s);
    switch (mode) {
        case GM_STORE: return split ? hipErrorInvalidValue : go_big<GM_STORE, M3, GR_DENSE, 1>(a, batch, s);
        case GM_RESID: return split ? go_big<GM_RESID, M3, GR_DENSE, 4>(a, batch, s) : go<GM_RESID, M3, GR_DENSE, 1>(a, batch, s);
        case GM_LINE: return split ? go_big<GM_LINE, M3, GR_DENSE, 4>(a, batch, s) : go_big<GM_LINE, M3, GR_DENSE, 1>(a, batch, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int gemm_partial_slots(int M, int N) { return ((M + 31) / 32) * ((N + 31) / 32); }

hipError_t launch_cgemm(int mode, const GemmArgs &a0, int batch, hipStream_t s, int role, bool m3, bool split) {
    GemmArgs a = a0;
    const int wt = split ? 32 : 64;
    if (a.M <= 0 || a.N <= 0 || batch <= 0) return hipSuccess;
    if (role < GR_DENSE || role > GR_ADJOINT) return hipErrorInvalidValue;
    const bool stage = role == GR_TILE || role == GR_TILE_TA_CB;
    const bool ta = role == GR_TILE_TA_CB || role == GR_ADJOINT;
    if (a.M % 64 || a.N % 64 || a.K % GEMM_BK || a.K <= 0) return hipErrorInvalidValue;   // padded operands only
    if ((ta && mode != GM_STORE) || (stage && (split || !m3))) return hipErrorInvalidValue;
    if (mode == GM_STORE && role == GR_DENSE && !a.cmap) return hipErrorInvalidValue;
    if (a.K2 < 0 || a.K2 > a.K || a.K2 % GEMM_BK || (a.K2 && !(mode == GM_LINE && stage))) return hipErrorInvalidValue;
    if (a.nz3 > 1 || a.nz4 > 1) {
        const int64_t inner = (int64_t)std::max(1, a.nz3) * std::max(1, a.nz4);
        if (!(mode == GM_STORE && stage && a.nz2 > 1 && a.nz2 % inner == 0)) return hipErrorInvalidValue;
    }
    if (a.scat_kp < 0 || (a.scat_kp && (!(mode == GM_STORE && stage) || a.scat_w < a.scat_kp || a.scat_lim <= 0 ||
                                        a.scat_lim > a.N)))
        return hipErrorInvalidValue;
    a.tiles_m = a.M / wt;
    a.tiles_n = a.N / wt;
    a.Mt = a.Mt > 0 ? std::min(a.Mt, a.M) : a.M;
    a.Nt = a.Nt > 0 ? std::min(a.Nt, a.N) : a.N;
    if (ta && a.lda < a.Mt) return hipErrorInvalidValue;
    a.b2_off = mode == GM_LINE ? a.B2 - a.B : 0;
    if (a.b2_off < 0) return hipErrorInvalidValue;
    const Extents ex = gemm_extents(a.M, a.N, a.K, a.Mt, a.Kt > 0 ? std::min(a.Kt, a.K) : a.K, ta, a.lda, a.ldb, a.b2_off);
    if (!ex.fit) return hipErrorInvalidValue;
    a.bytesA = ex.bytesA;
    a.bytesB = ex.bytesB;
    if (!stage) return m3 ? go_dense<true>(mode, a, batch, s, role, split) : go_dense<false>(mode, a, batch, s, role, split);
    if (role == GR_TILE_TA_CB) return go_big<GM_STORE, true, GR_TILE_TA_CB, 1>(a, batch, s);
    switch (mode) {
        case GM_STORE: return go_big<GM_STORE, true, GR_TILE, 1>(a, batch, s);
        case GM_RESID: return go<GM_RESID, true, GR_TILE, 1>(a, batch, s);
        case GM_LINE: return go<GM_LINE, true, GR_TILE, 1>(a, batch, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tlr
