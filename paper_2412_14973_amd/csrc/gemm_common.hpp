// Shared pieces of the complex GEMM kernels (FP32 and BF16 hi+lo split):
// the accumulator layout of the 32 x 32 MFMA blocks and the epilogue.
#pragma once
#include "common.hpp"

namespace tlr {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Output layout of a 32x32 MFMA accumulator (f32 result of the 32x32x2 f32 and
// 32x32x16 bf16 instructions): lane l holds column l % 32, register r holds
// row (r % 4) + 8 (r / 4) + 4 (l / 32).
__device__ __forceinline__ int acc_row(int r, int lane) {
    return (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// a uniform pointer, in scalar registers: where the compiler has computed it in vector registers, every buffer load
// from it would become a loop over the lanes' values
__device__ __forceinline__ void *scalar(const void *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return reinterpret_cast<void *>(lo | hi << 32);
}

// one component's products of the line-search sums: Re<r,a>, |a|^2, Re<r,b>, Re<a,b>, |b|^2
__device__ __forceinline__ void line_terms(float (&blk)[5], float r, float a, float b) {
    blk[0] = fmaf(r, a, blk[0]);
    blk[1] = fmaf(a, a, blk[1]);
    blk[2] = fmaf(r, b, blk[2]);
    blk[3] = fmaf(a, b, blk[3]);
    blk[4] = fmaf(b, b, blk[4]);
}

// One batch entry's epilogue operands.
struct EpiArgs {
    float2 *C, *C2;    // output; GM_LINE: a and b
    int64_t ldc;
    const float2 *E;   // GM_RESID: U (true shape Me x Ne); GM_LINE: r
    int64_t lde;
    int32_t Me, Ne;
    int32_t Mc, Nc;    // C is stored inside Mc x Nc only (not GM_LINE)
    double *partials;
    int32_t nblk;      // 32-column blocks of C per row of blocks (partial slots are numbered by block)
    const int64_t *cmap;                 // GM_STORE with COL_MAP (see GemmArgs)
    int32_t scat_kp, scat_w, scat_lim;   // GM_STORE with COL_SCAT: column scatter of the tile stages (see GemmArgs)
    int64_t scat_js;
};
enum ColumnsOfC { COL_PLAIN, COL_SCAT, COL_MAP };

// Epilogue of a wave's HB x CB blocks of 32 x 32 complex entries from row m0 and column n0 on, each lane holding
// whole entries of column lane % 32: cval(h, n, r) is accumulator row r of row block h and block n (GM_LINE: n = 0
// is a and n = 1 is b at the same columns). GM_STORE: C = AB. GM_RESID: C = AB - E and the sum of |C|^2. GM_LINE:
// the five line sums. KS > 1: the workgroup's KS waves hold shares of the same blocks; they are added in LDS in a
// fixed order, each wave finishing 16 / KS rows of every lane. A block's sums are its lanes' FP32 sums over the
// rows, real and imaginary parts apart (16 products at most), added in FP64, one partial slot per 32 x 32 block,
// numbered by block row and column whatever the tile.
// GM_RESID: also(h, cb, v) gets the finished rows of a lane (KS > 1: rows wave * 16 / KS and on of its registers).
struct Nothing {
    template <class V>
    __device__ __forceinline__ void operator()(int, int, const V &) const {}
};
template <int MODE, int COLS, int KS, int HB, int CB, class F, class G = Nothing>
__device__ __forceinline__ void block_epilogue(const EpiArgs &ea, F &&cval, int m0, int n0, G &&also = G()) {
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int col = n0 + (lane & 31);
    constexpr int NR = 16 / KS;                   // rows of a block that this wave finishes
    constexpr int NS = MODE == GM_RESID ? 1 : 5;
    constexpr int NV = MODE == GM_LINE ? 2 : 1;   // a and b, or one block of C
    auto row_of = [&](int h, int r) { return m0 + 32 * h + acc_row(KS == 1 ? r : wave * NR + r, lane); };
    __shared__ float2 part[KS][KS == 1 ? 1 : 16][KS == 1 ? 1 : 64];   // one block at a time: less LDS, more waves
    __shared__ double red[KS][NS];
#pragma unroll
    for (int h = 0; h < HB; ++h)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int cc = col + 32 * cb;
            // two loops: a condition on every store costs the full blocks a fifth of the whole product
            const bool whole = m0 + 32 * h + 32 <= ea.Mc && n0 + 32 * cb + 32 <= ea.Nc;
            auto put = [&](int64_t ccol, const float2 (&c)[NR]) {
                if (whole) {
#pragma unroll
                    for (int r = 0; r < NR; ++r) ea.C[(int64_t)row_of(h, r) * ea.ldc + ccol] = c[r];
                } else if (cc < ea.Nc) {
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if (row_of(h, r) < ea.Mc) ea.C[(int64_t)row_of(h, r) * ea.ldc + ccol] = c[r];
                }
            };
            // the entries of E: their loads are in flight together, and during the sums over the waves (an
            // entry outside E reads E[0] and is dropped)
            float2 e[NR];
            if constexpr (MODE != GM_STORE) {
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const int row = row_of(h, r);
                    const bool in = MODE == GM_LINE || (row < ea.Me && cc < ea.Ne);
                    e[r] = ea.E[in ? (int64_t)row * ea.lde + cc : 0];
                    if (!in) e[r] = make_float2(0.f, 0.f);
                }
            }
            float2 v[NV][NR];
#pragma unroll
            for (int n = 0; n < NV; ++n) {
                if constexpr (KS == 1) {
#pragma unroll
                    for (int r = 0; r < NR; ++r) v[n][r] = cval(h, MODE == GM_LINE ? n : cb, r);
                } else {
                    if (h + cb + n) __syncthreads();   // the block before is finished
#pragma unroll
                    for (int r = 0; r < 16; ++r) part[wave][r][lane] = cval(h, MODE == GM_LINE ? n : cb, r);
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        float2 s = part[0][wave * NR + r][lane];
#pragma unroll
                        for (int w = 1; w < KS; ++w) {
                            const float2 x = part[w][wave * NR + r][lane];
                            s.x += x.x;
                            s.y += x.y;
                        }
                        v[n][r] = s;
                    }
                }
            }
            float blk[2][NS];
#pragma unroll
            for (int q = 0; q < NS; ++q) blk[0][q] = blk[1][q] = 0.f;
            if constexpr (MODE == GM_STORE) {
                int64_t ccol = cc;
                if (COLS == COL_SCAT && ea.scat_kp > 0) {
                    if (cc >= ea.scat_lim) continue;
                    ccol += (int64_t)((cc % ea.scat_w) / ea.scat_kp) * ea.scat_js;
                }
                if (COLS == COL_MAP) {
                    ccol = ea.cmap[cc];
                    if (ccol < 0) continue;
                }
                put(ccol, v[0]);
            } else if constexpr (MODE == GM_RESID) {
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    // zero outside E: an operand read in place has other entries there than zeros
                    const bool in = row_of(h, r) < ea.Me && cc < ea.Ne;
                    const float2 d = in ? make_float2(v[0][r].x - e[r].x, v[0][r].y - e[r].y) : make_float2(0.f, 0.f);
                    blk[0][0] = fmaf(d.x, d.x, blk[0][0]);
                    blk[1][0] = fmaf(d.y, d.y, blk[1][0]);
                    v[0][r] = d;
                }
                put(cc, v[0]);
                also(h, cb, v[0]);
            } else {
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    ea.C[(int64_t)row_of(h, r) * ea.ldc + cc] = v[0][r];
                    ea.C2[(int64_t)row_of(h, r) * ea.ldc + cc] = v[NV - 1][r];
                    line_terms(blk[0], e[r].x, v[0][r].x, v[NV - 1][r].x);
                    line_terms(blk[1], e[r].y, v[0][r].y, v[NV - 1][r].y);
                }
            }
            if constexpr (MODE != GM_STORE) {
                const int64_t slot = (int64_t)((m0 >> 5) + h) * ea.nblk + (cc >> 5);
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    const double s = wave_sum((double)blk[0][q] + (double)blk[1][q]);
                    if (lane == 0) {
                        if constexpr (KS == 1) ea.partials[slot * NS + q] = s;
                        else red[wave][q] = s;
                    }
                }
                if constexpr (KS > 1) {
                    static_assert(KS == 4, "the fixed order of the waves' sums");
                    __syncthreads();
                    if (t < NS) ea.partials[slot * NS + t] = (red[0][t] + red[1][t]) + (red[KS - 2][t] + red[KS - 1][t]);
                }
            }
        }
}

}  // namespace tlr
