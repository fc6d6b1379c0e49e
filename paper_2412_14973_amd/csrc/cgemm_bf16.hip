// Complex64 GEMM on CDNA4 BF16 matrix cores with a hi+lo split.
//
// Every FP32 operand x is carried as two BF16 numbers, hi = bf16(x) and
// lo = bf16(x - hi); a product is evaluated as lo*hi + hi*lo + hi*hi with FP32
// accumulation (the lo*lo term, about 2^-16 of the product, is dropped).
// A is M x K complex, B is given TRANSPOSED, N x K complex ("NT" form); for the
// products of the method this is free: X, X1 and X2 are symmetric, and r^T is
// written by the kernel that updates r. Operands are pre-split into separate hi
// and lo planes of interleaved complex BF16 (4 bytes per complex). A row of A is
// then a real row (Re, Im, Re, Im, ...); the real part of C takes the B row with
// its imaginary parts negated (one XOR per word), the imaginary part the row with
// (Re, Im) swapped (one rotation per word). One v_mfma_f32_32x32x16_bf16
// multiplies 8 complex k of one of these products.
//
// As in cgemm.hip, every wave feeds its matrix instructions from global memory
// through registers, without LDS and without a barrier in the k loop, here with
// 2 x 2 blocks of 32 x 32 complex entries per wave (GM_LINE: two row blocks of a
// and b): one block per wave asks L1 for 85 bytes per cycle and CU at the matrix
// cores' rate, which is more than its 64; four ask for 43. The planes hold the
// operands in the order of these loads (plane_word), which is what makes this work:
// from row-major planes the same kernel reads 32 bytes of each cache line at a time
// and reaches 235 of 424 Tflop/s (64 problems of 1024^2). The next chunk's loads are in flight during a chunk's products: 5 to 10 %.
// What bounds it: at 4096^2 463 to 476 Tflop/s of complex products (8 m n k), that is 1.4 Pflop/s of
// BF16 products, above what a library product of 8192^3 reaches (1.04). Before, with 256 x 128 tiles
// fed through LDS: 367 to 403, and at 1024^2 32 tiles for 256 CUs.
// us for r = D X - U, D^H r and [a | b] (the first writes r^T's planes too, which took a pass of its own before):
//   nr = ns     64 x 8 problems   448            1024            2304            1024 x 64 problems
//   before      33, 15, 19        95, 60, 64     162, 127, 133   346, 295, 656   1953, 1446, 2948
//   now         7, 7, 8           10, 9, 12      32, 26, 49      251, 237, 450   1403, 1206, 2468
#include <algorithm>

#include "gemm_common.hpp"

namespace tlr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

namespace {

template <int HB, int NB>
struct Chunk {
    u32x4 a[HB][2], b[NB][2];   // [block][hi, lo]: 4 complex k per lane, lane half h holding 4 h .. 4 h + 3
};

template <int MODE, int HB, int CB, int KS>
__global__ __launch_bounds__(256, 2) void cgemm_bf16x3_kernel(GemmArgsB g) {
    constexpr int NB = MODE == GM_LINE ? 2 : CB;   // column blocks of B (GM_LINE: of X1 and of X2)
    constexpr int WV = KS == 1 ? 2 : 1;            // waves per workgroup tile row and column
    const int z = blockIdx.y;
    // contiguous tile ranges per XCD, grouped by 8 tile rows
    const int nwg = gridDim.x;
    int pid = blockIdx.x;
    if ((nwg & 7) == 0) pid = (pid & 7) * (nwg >> 3) + (pid >> 3);
    const int per_group = 8 * g.tiles_n;
    const int grp = pid / per_group;
    const int gsz = min(g.tiles_m - 8 * grp, 8);
    const int tm = 8 * grp + (pid % per_group) % gsz;
    const int tn = (pid % per_group) / gsz;

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m0 = 32 * HB * (tm * WV + (KS == 1 ? wave >> 1 : 0));
    const int n0 = 32 * CB * (tn * WV + (KS == 1 ? wave & 1 : 0));

    __amdgpu_buffer_rsrc_t rsA[2], rsB[2];
    rsA[0] = __builtin_amdgcn_make_buffer_rsrc(scalar(g.Ahi + z * g.sA), (short)0, (int)g.bytesA, 0x00020000);
    rsA[1] = __builtin_amdgcn_make_buffer_rsrc(scalar(g.Alo + z * g.sA), (short)0, (int)g.bytesA, 0x00020000);
    rsB[0] = __builtin_amdgcn_make_buffer_rsrc(scalar(g.Bhi + z * g.sB), (short)0, (int)g.bytesB, 0x00020000);
    rsB[1] = __builtin_amdgcn_make_buffer_rsrc(scalar(g.Blo + z * g.sB), (short)0, (int)g.bytesB, 0x00020000);
    uint32_t offA[HB], offB[NB];
#pragma unroll
    for (int h = 0; h < HB; ++h) offA[h] = (uint32_t)((m0 + 32 * h) * (g.lda * 4)) + lane * 16;
#pragma unroll
    for (int n = 0; n < NB; ++n)
        offB[n] = (uint32_t)((n0 + n * (MODE == GM_LINE ? g.b2_rows : 32)) * (g.ldb * 4)) + lane * 16;

    auto load = [&](Chunk<HB, NB> &c, int kt) {
        const int so = kt * 1024;   // one block of a plane
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
            for (int h = 0; h < HB; ++h) c.a[h][p] = __builtin_amdgcn_raw_buffer_load_b128(rsA[p], (int)offA[h], so, 0);
#pragma unroll
            for (int n = 0; n < NB; ++n) c.b[n][p] = __builtin_amdgcn_raw_buffer_load_b128(rsB[p], (int)offB[n], so, 0);
        }
    };

    floatx16 acc[HB][NB][2];   // real and imaginary part
#pragma unroll
    for (int h = 0; h < HB; ++h)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[h][n][p][r] = 0.f;

    auto mfma = [](u32x4 a, u32x4 b, floatx16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    };
    auto compute = [&](const Chunk<HB, NB> &c) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            u32x4 b[2][2];   // [hi, lo][for the real, for the imaginary part]
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    b[p][0][w] = c.b[n][p][w] ^ 0x80000000u;
                    b[p][1][w] = __builtin_amdgcn_alignbit(c.b[n][p][w], c.b[n][p][w], 16);
                }
#pragma unroll
            for (int q = 0; q < 3; ++q)   // lo hi, hi lo, hi hi
#pragma unroll
                for (int h = 0; h < HB; ++h)
#pragma unroll
                    for (int p = 0; p < 2; ++p) acc[h][n][p] = mfma(c.a[h][q == 0 ? 1 : 0], b[q == 1 ? 1 : 0][p], acc[h][n][p]);
        }
    };

    const int nk = m0 < g.Mt && n0 < g.Nt ? g.K / PLANE_KB : 0;
    int kt = KS == 1 ? 0 : wave;
    Chunk<HB, NB> r0, r1;
    if (kt < nk) {
        // the next chunk's loads without a branch around them (the last one's again at the end): behind a branch
        // that may have skipped them, the wait for the chunk at hand would be a wait for all
        load(r0, kt);
        for (; kt + KS < nk; kt += 2 * KS) {
            load(r1, kt + KS);
            __builtin_amdgcn_sched_barrier(0);
            compute(r0);
            load(r0, min(kt + 2 * KS, nk - 1));
            __builtin_amdgcn_sched_barrier(0);
            compute(r1);
        }
        if (kt < nk) compute(r0);
    }

    EpiArgs ea;
    ea.C = g.C + z * g.sC;
    ea.C2 = MODE == GM_LINE ? g.C2 + z * g.sC : nullptr;
    ea.ldc = g.ldc;
    ea.E = MODE == GM_STORE ? nullptr : g.E + z * g.sE;
    ea.lde = g.lde;
    ea.Me = g.Me;
    ea.Ne = g.Ne;
    ea.Mc = g.Mc;
    ea.Nc = g.Nc;
    ea.partials = g.partials ? g.partials + z * g.sP : nullptr;
    ea.nblk = g.N >> 5;
    // four registers of a lane are 16 bytes of C^T's split planes, at this lane's place in a block
    uint32_t *const Thi = MODE == GM_RESID && g.Thi ? g.Thi + z * g.sT : nullptr;
    uint32_t *const Tlo = Thi ? g.Tlo + z * g.sT : nullptr;
    auto put_t = [&](int h, int cb, const float2 (&v)[16 / KS]) {
        if (!Thi) return;
        const int64_t w0 = plane_word(n0 + 32 * cb, m0 + 32 * h, g.ldt) + (KS > 1 ? wave * 256 : 0) + lane * 4;
#pragma unroll
        for (int q = 0; q < 4 / KS; ++q) {
            uint4 hi, lo;
            split_c(v[4 * q], hi.x, lo.x);
            split_c(v[4 * q + 1], hi.y, lo.y);
            split_c(v[4 * q + 2], hi.z, lo.z);
            split_c(v[4 * q + 3], hi.w, lo.w);
            *reinterpret_cast<uint4 *>(Thi + w0 + 256 * q) = hi;
            *reinterpret_cast<uint4 *>(Tlo + w0 + 256 * q) = lo;
        }
    };
    block_epilogue<MODE, COL_PLAIN, KS, HB, CB>(
        ea, [&](int h, int n, int r) { return make_float2(acc[h][n][0][r], acc[h][n][1][r]); }, m0, n0, put_t);
}

template <int MODE, int HB, int CB, int KS>
hipError_t go(GemmArgsB a, int batch, hipStream_t s) {
    constexpr int WV = KS == 1 ? 2 : 1;
    if (a.M % (32 * HB * WV) || a.N % (32 * CB * WV)) return hipErrorInvalidValue;
    a.tiles_m = a.M / (32 * HB * WV);
    a.tiles_n = a.N / (32 * CB * WV);
    hipLaunchKernelGGL((cgemm_bf16x3_kernel<MODE, HB, CB, KS>), dim3(a.tiles_m * a.tiles_n, batch), dim3(256), 0, s, a);
    return hipGetLastError();
}

// A wave takes two by two blocks where every CU gets a workgroup of such tiles: 4 problems of 448^2 (196 tiles)
// 24, 17, 28 us against 20, 17, 29 with one block per wave, one of 1024^2 (256) 35, 29, 51 against 34, 31, 54,
// of 2304 x 576 (324) 85, 71, 134 against 87, 77, 147, of 2304^2 (1296) 262, 246, 469 against 298, 292, 506 (all
// before the loads of a chunk were moved ahead of the products of the last).
constexpr int64_t BIG_TILES = 256;

template <int MODE>
hipError_t pick(const GemmArgsB &a, int batch, hipStream_t s, bool split) {
    constexpr int CB = MODE == GM_LINE ? 1 : 2;
    if (!split) return go<MODE, 2, CB, 1>(a, batch, s);
    const int64_t tiles = (int64_t)((a.Mt + 63) / 64) * ((a.Nt + 63) / 64) * batch;
    return tiles >= BIG_TILES ? go<MODE, 2, CB, 4>(a, batch, s) : go<MODE, 1, 1, 4>(a, batch, s);
}

}  // namespace

hipError_t launch_cgemm_bf16(int mode, const GemmArgsB &a0, int batch, hipStream_t s, bool split) {
    GemmArgsB a = a0;
    if (a.M <= 0 || a.N <= 0 || batch <= 0) return hipSuccess;
    if (a.M % GEMM_PAD || a.N % GEMM_PAD || a.K % 32 || a.K <= 0 || a.lda % PLANE_KB ||
        a.ldb % PLANE_KB || (mode == GM_LINE && a.b2_rows % 32)) return hipErrorInvalidValue;   // padded operands only
    a.Mt = a.Mt > 0 ? std::min(a.Mt, a.M) : a.M;
    a.Nt = a.Nt > 0 ? std::min(a.Nt, a.N) : a.N;
    const int64_t bytesA = (int64_t)a.M * a.lda * 4;
    const int64_t rowsB = (mode == GM_LINE) ? a.b2_rows + a.N : a.N;
    const int64_t bytesB = rowsB * a.ldb * 4;
    if (bytesA >= (int64_t)1 << 32 || bytesB >= (int64_t)1 << 32) return hipErrorInvalidValue;
    a.bytesA = (uint32_t)bytesA;
    a.bytesB = (uint32_t)bytesB;
    switch (mode) {
        case GM_STORE: return pick<GM_STORE>(a, batch, s, split);
        case GM_RESID: return pick<GM_RESID>(a, batch, s, split);
        case GM_LINE: return pick<GM_LINE>(a, batch, s, split);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tlr
