// Tile kernels: assembly of X = C(Zbar, Lbar, Rbar) and the per-tile gradient
// contractions.
//
// Assembly (Tile Low-rank MDD section): X_ij = L_ij R_ij for i > j and
// X_ji = X_ij^T; X_ii = Q_ii Q_ii^T or (Z_ii + Z_ii^T)/2. The directional
// form used by the exact line search expands C(theta + a p) = C(theta) +
// a X1 + a^2 X2, tile by tile: X1 = P_L R + L P_R, X2 = P_L P_R (and the
// Q Q^T / dense analogues). Each workgroup builds one 64 x 64 block on the
// FP32 matrix cores from factors staged in LDS 16 rank entries at a time;
// every product is staged through LDS once and written from there twice
// (directly and transposed, both with whole rows per wave), so X = X^T holds
// bit for bit; Q Q^T tiles are built on and below the block diagonal only
// and mirrored.
//
// Gradient (ADMM solver section, eqs. DXLR): with W = D^H r and W' = W + W^T,
// grad L = W' R^H, grad R = L^H W', grad Q = W' conj(Q), grad Z = W'/2.
// W' is never formed: its entries are added in registers from W_ij and W_ji.
#include <type_traits>

#include "gemm_common.hpp"

namespace tlr {
namespace {

// Output: complex64 (OUTB = false) or split BF16 planes (OUTB = true, see launch_assemble).
template <bool OUTB>
__device__ __forceinline__ void put(float2 *X, int64_t row, int64_t col, int64_t ldx, int64_t low, float2 v) {
    if (OUTB) {
        uint32_t h, l;
        split_c(v, h, l);
        uint32_t *w = reinterpret_cast<uint32_t *>(X) + plane_word(row, col, ldx);
        w[0] = h;
        w[low] = l;
    } else {
        X[row * ldx + col] = v;
    }
}
// entry e of a 64 x 64 block in the order of the output: along its rows, or four entries of each row in turn; and how
// many of them reach the last of the block's true rows and columns (the blocks of small tiles are mostly empty)
template <bool OUTB>
__device__ __forceinline__ void out_entry(int e, int &row, int &col) {
    row = OUTB ? (e >> 2) & 63 : e >> 6;
    col = OUTB ? ((e >> 8) << 2) + (e & 3) : e & 63;
}
template <bool OUTB>
__device__ __forceinline__ int out_entries(int rows, int cols) {
    return OUTB ? (cols + 3) / 4 * 256 : rows * 64;
}


typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t OUTSIDE = 0xffffff00u;   // a buffer offset past every end

constexpr int AB = ASM_B;            // block edge (rows and columns)
constexpr int AKC = ASM_KC;          // rank entries staged per step
constexpr int AAP = AB + 1;          // row-factor planes [AKC][AAP] floats (k-major: rows fastest)
constexpr int ABP = AB + 1;          // column-factor stage [AKC][ABP] complex
constexpr int ST_P = AB + 1;         // transpose stage [AB][ST_P] complex
constexpr int A_PL = AKC * AAP;      // floats per row-factor plane
constexpr int B_ST = AKC * ABP;      // complex per column-factor stage

// Each workgroup builds one 64 x 64 block of a tile on the FP32 matrix cores. A factor product
// F G (F: 64 x k rows of L, P_L or Q; G: k x 64 columns of R, P_R or Q^T) is a complex GEMM with
// K = k, evaluated in realified form: one v_mfma_f32_32x32x2_f32 per complex k takes (Re, Im) of
// F[m][k] as its two A entries and the real 2 x 2 block [[Re g, Im g], [-Im g, Re g]] of G[k][n] as
// B, so the real output columns come out as interleaved (re, im) pairs. Wave w owns complex columns
// 16 w .. 16 w + 15 of the block and both 32-row halves: X (or X1 and X2) in two (four) accumulators.
// The row factors sit in LDS as separate real and imaginary planes, k-major, so a lane's A entry
// is one conflict-free float read; the column factors stay interleaved complex. 33 KB of LDS and
// at most 128 VGPRs (launch bound: 4 waves per SIMD) keep four workgroups on a CU, so the write
// phases of some overlap the loads and products of others. The latency of the phases is what bounds it, so a chunk's
// loads are in flight together, and so are the LDS reads of whole blocks before their stores: us of 8 problems of nr
// 1024 (k 25 to 48) X 48.6 with a condition at each, 34.7 with the loads so, 33.1 with both, [X1 | X2] 81.8, 67.9 and
// 66.4 (its writes take 26, its products 54), X in BF16 planes of nr 2304 33.6 and 30.3 (loads, both). A chunk ahead
// during the products takes registers that spill: 71.7.
template <bool DIR, bool OUTB>
__global__ __launch_bounds__(256, 4) void assemble_kernel(const TileDesc *__restrict__ tiles,
                                                       const AsmItem *__restrict__ items,
                                                       const ProbOff *__restrict__ probs,
                                                       const float2 *__restrict__ theta_base,
                                                       const float2 *__restrict__ p_base,
                                                       float2 *__restrict__ X_base,
                                                       float2 *__restrict__ X2_base,
                                                       int64_t x2w, int64_t low) {
    constexpr int NF = DIR ? 2 : 1;   // factor sets: (L, R) and, for the directional form, (P_L, P_R)
    constexpr int SA_F = NF * 2 * A_PL;                 // floats
    constexpr int SB_F = NF * 2 * B_ST;                 // floats
    constexpr int ST_F = 2 * AB * ST_P;
    constexpr int SM_F = (SA_F + SB_F > ST_F) ? SA_F + SB_F : ST_F;
    __shared__ float smem[SM_F];
    float *sA = smem;                                  // [NF][re, im][AKC][AAP]
    float2 *sB = reinterpret_cast<float2 *>(smem + SA_F);   // [NF][AKC][ABP]
    float2 *sT = reinterpret_cast<float2 *>(smem);     // transpose stage, reused after the k loop

    const AsmItem it = items[blockIdx.x];
    const TileDesc td = tiles[it.tile];
    const ProbOff po = probs[it.prob];
    const float2 *theta = theta_base + po.theta;
    const float2 *pv = DIR ? p_base + po.theta : nullptr;
    // complex64: X at element po.x; split planes: X hi plane at word 2 po.x, X2 at + x2w words
    float2 *X = OUTB ? reinterpret_cast<float2 *>(reinterpret_cast<uint32_t *>(X_base) + 2 * po.x) : X_base + po.x;
    float2 *X2 = !DIR ? nullptr
                      : (OUTB ? reinterpret_cast<float2 *>(reinterpret_cast<uint32_t *>(X_base) + 2 * po.x + x2w)
                              : X2_base + po.x);
    const int64_t ldx = po.ldx;

    const int t = threadIdx.x;
    const int r0 = it.r0, c0 = it.c0;
    const int nrow = min(AB, td.di - r0);
    const int ncol = min(AB, td.dj - c0);

    if (td.kind == TILE_DENSE) {
        // X = (Z + Z^T)/2 ; X1 = (P + P^T)/2 ; X2 = 0 (element-wise, no products)
        const float2 *Z = DIR ? pv + td.offA : theta + td.offA;
        const int d = td.di;
        for (int e = t; e < AB * AB; e += 256) {   // transposed block Z[c0+cc][r0+rr]
            const int cc = e >> 6, rr = e & 63;
            float2 v = make_float2(0.f, 0.f);
            if (cc < ncol && rr < nrow) v = Z[(int64_t)(c0 + cc) * d + r0 + rr];
            sT[cc * ST_P + rr] = v;
        }
        __syncthreads();
        for (int e = t; e < AB * AB; e += 256) {
            int rr, cc;
            out_entry<OUTB>(e, rr, cc);
            if (rr < nrow && cc < ncol) {
                const float2 zd = Z[(int64_t)(r0 + rr) * d + c0 + cc];
                const float2 zt = sT[cc * ST_P + rr];
                const int64_t row = td.row0 + r0 + rr, col = td.col0 + c0 + cc;
                put<OUTB>(X, row, col, ldx, low, make_float2(0.5f * (zd.x + zt.x), 0.5f * (zd.y + zt.y)));
                if (DIR) put<OUTB>(X2, row, col, ldx, low, make_float2(0.f, 0.f));
            }
        }
        return;
    }

    const int lane = t & 63, wave = t >> 6;
    const int j32 = lane & 31, half = lane >> 5;
    const int cb = 16 * wave;                                   // first complex column of the wave
    const int bidx = 2 * cb + (j32 ^ half);                     // float of the realified B entry
    const uint32_t bsign = (half && !(j32 & 1)) ? 0x80000000u : 0u;   // -Im g in the second k row

    floatx16 acc[2][2];   // [X | X1, X2][row half]
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][i][r] = 0.f;

    const bool qq = (td.kind == TILE_QQ);
    const int k = td.k;
    const float2 *Lf = theta + td.offA;                 // L (di x k) or Q (d x k)
    const float2 *Rf = qq ? Lf : theta + td.offB;       // R (k x dj) or Q again
    const float2 *PLf = DIR ? pv + td.offA : nullptr;
    const float2 *PRf = DIR ? (qq ? PLf : pv + td.offB) : nullptr;
    // A chunk of the factors: an entry outside them is past its buffer's end and reads zero, so the loads carry no
    // conditions and are in flight together. A factor Q can hold 4 GiB and more, so offsets count from the block's first
    // row (of R: column).
    constexpr int NE = AB * AKC / 256;
    auto buffer = [&](const float2 *p, uint32_t entries) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float2 *>(p), (short)0, (int)(8u * entries), 0x00020000);
    };
    const int64_t oL = (int64_t)r0 * k, oR = qq ? (int64_t)c0 * k : c0;
    const uint32_t nL = (uint32_t)nrow * k, nR = qq ? (uint32_t)ncol * k : (uint32_t)k * td.dj - c0;
    const auto La = buffer(Lf + oL, nL), Ra = buffer(Rf + oR, nR);
    const auto Pl = buffer((DIR ? PLf : Lf) + oL, nL), Pr = buffer((DIR ? PRf : Rf) + oR, nR);
    u32x2 va[NE][NF], vb[NE][NF];
    auto load = [&](int kc0) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = t + 256 * i;
            // row factors: rows r0.., k contiguous in theta; column factors G[kk][cc] = R[kc0+kk][c0+cc] or
            // Q[c0+cc][kc0+kk]
            const int rr = e / AKC, kr = kc0 + e % AKC;
            const int cc = qq ? e / AKC : e & 63, kk = kc0 + (qq ? e % AKC : e >> 6);
            const uint32_t oa = rr < nrow && kr < k ? 8u * (uint32_t)(rr * k + kr) : OUTSIDE;
            const uint32_t ob = cc < ncol && kk < k ? 8u * (uint32_t)(qq ? cc * k + kk : kk * td.dj + cc) : OUTSIDE;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                va[i][f] = __builtin_amdgcn_raw_buffer_load_b64(f ? Pl : La, (int)oa, 0, 0);
                vb[i][f] = __builtin_amdgcn_raw_buffer_load_b64(f ? Pr : Ra, (int)ob, 0, 0);
            }
        }
    };
    for (int kc0 = 0; kc0 < k; kc0 += AKC) {
        const int kn = min(AKC, k - kc0);
        load(kc0);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = t + 256 * i;
            const int cc = qq ? e / AKC : e & 63, kk = qq ? e % AKC : e >> 6;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                float *pl = sA + f * 2 * A_PL + e % AKC * AAP + e / AKC;
                pl[0] = __uint_as_float(va[i][f].x);
                pl[A_PL] = __uint_as_float(va[i][f].y);
                sB[f * B_ST + kk * ABP + cc] = make_float2(__uint_as_float(vb[i][f].x), __uint_as_float(vb[i][f].y));
            }
        }
        __syncthreads();
        const float *bf = reinterpret_cast<const float *>(sB);
        for (int kk = 0; kk < kn; ++kk) {
            float a[NF][2], b[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
#pragma unroll
                for (int i = 0; i < 2; ++i) a[f][i] = sA[f * 2 * A_PL + half * A_PL + kk * AAP + 32 * i + j32];
                b[f] = __uint_as_float(__float_as_uint(bf[2 * (f * B_ST + kk * ABP) + bidx]) ^ bsign);
            }
            if (!DIR) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][i], b[0], acc[0][i], 0, 0, 0);
            } else {
                // X1 += P_L R + L P_R ; X2 += P_L P_R (the two X1 products of a row half three apart)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[NF - 1][i], b[0], acc[0][i], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[1][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[NF - 1][i], b[NF - 1], acc[1][i], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][i], b[NF - 1], acc[0][i], 0, 0, 0);
            }
        }
        __syncthreads();
    }

    // Lane (j32, half) holds component j32 & 1 of complex column cb + j32 / 2 for rows
    // acc_row(r, lane) (+ 32 for the second half). Each product is staged through LDS once and
    // written from there twice, both times with whole rows per wave: X_ij directly and X_ji = X_ij^T.
    // Q Q^T tiles are built on and below the block diagonal only and mirrored, so the tile is
    // symmetric bit for bit: direct write where row >= column, transposed write where row > column.
    const int ccol = cb + (j32 >> 1);
    const int comp = j32 & 1;
    float *sTf = smem;   // [row][ST_P] complex
    const bool whole = nrow == AB && ncol == AB && (!qq || r0 != c0);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sTf[2 * ((32 * i + acc_row(r, lane)) * ST_P + ccol) + comp] = acc[f][i][r];
        __syncthreads();
        float2 *dst = f ? X2 : X;
        if (whole) {   // no conditions: the reads of several entries are in flight together
#pragma unroll 8
            for (int e = t; e < AB * AB; e += 256) {
                int rr, cc;
                out_entry<OUTB>(e, rr, cc);
                put<OUTB>(dst, td.row0 + r0 + rr, td.col0 + c0 + cc, ldx, low, sT[rr * ST_P + cc]);
            }
#pragma unroll 8
            for (int e = t; e < AB * AB; e += 256) {
                int rr, cc;
                out_entry<OUTB>(e, cc, rr);
                put<OUTB>(dst, td.col0 + c0 + cc, td.row0 + r0 + rr, ldx, low, sT[rr * ST_P + cc]);
            }
            continue;
        }
        for (int e = t; e < out_entries<OUTB>(nrow, ncol); e += 256) {
            int rr, cc;
            out_entry<OUTB>(e, rr, cc);
            if (rr < nrow && cc < ncol && (!qq || r0 + rr >= c0 + cc))
                put<OUTB>(dst, td.row0 + r0 + rr, td.col0 + c0 + cc, ldx, low, sT[rr * ST_P + cc]);
        }
        for (int e = t; e < out_entries<OUTB>(ncol, nrow); e += 256) {
            int rr, cc;
            out_entry<OUTB>(e, cc, rr);
            if (cc < ncol && rr < nrow && (!qq || r0 + rr > c0 + cc))
                put<OUTB>(dst, td.col0 + c0 + cc, td.row0 + r0 + rr, ldx, low, sT[rr * ST_P + cc]);
        }
    }
}

// One gradient item: a 32 x kn block (kn <= 64 rank entries from b0) of G = W' conj(F), where
//   G_L: rows of the tile, F[c][kk] = R[kk][c]    (G_L = W' R^H, contraction over tile columns)
//   G_Q: rows of the tile, F[c][kk] = Q[c][kk]    (G_Q = (W + W^T) conj(Q))
//   G_R: cols of the tile, F[r][kk] = L[r][kk]    (G_R^T = W'^T conj(L), contraction over tile rows)
// with W' = W_ij + W_ji^T formed in registers: both parts are read where they lie, one along the lanes' own rows
// (16 bytes at a time), one across them (a row of 32 entries at a time). The contraction runs on the FP32 matrix
// cores: a v_mfma_f32_32x32x2_f32 takes the real parts of W'[m][c] for two c, another one their imaginary parts, against
// (Re, -Im) and (Im, Re) of F[c][n] as two real columns each, so a lane holds one component of 16 rows of a rank entry.
// The item's four waves take chunks of 8 c in turn and their sums are added in LDS at the end; until then a wave waits
// for nobody.
//
// What bounds it: the matrix cores in full launches, where a rank is padded to 16 (4096^2 of tiles 256, rank 32: 67 us,
// 128 TFLOP/s of 8 d d k a product), else the chain of chunks. Before, a workgroup of 64 rows staged W' and F in LDS,
// 4 c and three barriers at a time: 113 us; nr 1024 (tiles 128, rank 20) 43 us, now 7.7; nr 2304 (tiles 512,
// rank 40) 166, now 49.
constexpr int GR_CH = 8;               // contraction entries per chunk: four per half of a wave
constexpr int GR_FAR = 8192;           // contraction rows that 32-bit offsets span (of up to 2^16 entries each)
static_assert(GR_FAR % (4 * GR_CH) == 0, "each wave's share of the contraction goes on where it ended");
constexpr int GP_P = 66;               // partial blocks [4 waves][16][GP_P] floats
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int KQ>
struct GradChunk {
    float2 w1[4], w2[4], f[KQ][4];
};

template <int KQ, bool FROW>
__device__ __forceinline__ void grad_block(const GradItem &it, const TileDesc &td, const float2 *__restrict__ W,
                                           int64_t ldw, const float2 *__restrict__ theta, float2 *__restrict__ g,
                                           float *smem) {
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int j32 = lane & 31, half = lane >> 5;
    const int k = td.k, a0 = it.a0, b0 = it.b0;
    const int kn = min(GR_KK, k - b0);
    const bool colside = it.kind == G_R;
    const int nout = min(GR_ROWS, (colside ? td.dj : td.di) - a0);   // out-rows in this item
    const int ncon = colside ? td.di : td.dj;                        // contraction length
    // W'[m][c] = w1[m ldw + c] + w2[c ldw + m]. Buffer loads: an offset past the end gives zero, so the chunks at
    // the end of the contraction need no branch (a branch would make each load wait for the ones before it).
    // W and a factor Q can hold 4 GiB and more (the BF16 products' planes of X are half as large), so offsets of 32 bits
    // count from the item's first row and, where the contraction runs over rows, from the first of GR_FAR of them (a base
    // for every chunk took nr 1024 from 7.7 us to 8.3, nr 4096 from 66 to 71).
    const uint32_t ld8 = (uint32_t)ldw * 8, k8 = (uint32_t)k * 8;
    const int64_t row1 = (colside ? td.col0 : td.row0) + a0, col1 = colside ? td.row0 : td.col0;
    const int64_t row2 = col1, col2 = row1;
    const float2 *W1 = W + row1 * ldw + col1, *W2 = W + row2 * ldw + col2;
    const float2 *F = theta + (FROW ? td.offB : td.offA);
    auto buffer = [](const float2 *p, uint32_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(scalar(p), (short)0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
    };
    const uint32_t m = min(j32, nout - 1);   // rows and rank entries past the item repeat its last one and are dropped
    const uint32_t o1 = m * ld8 + 32 * half, o2 = 4 * half * ld8 + m * 8;
    const int comp = j32 & 1;
    uint32_t of[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        const uint32_t n = b0 + min(16 * q + (j32 >> 1), kn - 1);
        of[q] = FROW ? n * td.dj * 8 + 32 * half : n * 8 + 4 * half * k8;
    }
    floatx16 acc[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
    for (int far = 0; far < ncon; far += GR_FAR) {
        const int n = min(ncon - far, GR_FAR);   // entries of the contraction from far on
        const auto rsW1 = buffer(W1 + far, (uint32_t)nout * ld8 - (uint32_t)(col1 + far) * 8);
        const auto rsW2 = buffer(W2 + far * ldw, n * ld8);   // what lies past the last row reads zero
        const auto rsF = FROW ? buffer(F + far, k8 * (uint32_t)td.dj - 8 * far) : buffer(F + (int64_t)far * k, n * k8);
        auto load = [&](GradChunk<KQ> &x, int ch) {
            const uint32_t c = ch * GR_CH, row = min(ch * GR_CH, n);
#pragma unroll
            for (int i = 0; i < 4; i += 2) {   // the second entry may lie past the tile: dropped in compute()
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsW1, (int)(o1 + 8 * i), (int)(8 * row), 0);
                x.w1[i] = make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
                x.w1[i + 1] = make_float2(__uint_as_float(v[2]), __uint_as_float(v[3]));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rsW2, (int)(o2 + i * ld8), (int)(row * ld8), 0);
                x.w2[i] = make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
                const bool in = !FROW || (int)c + 4 * half + i < n;   // past a row of R its next one follows
#pragma unroll
                for (int q = 0; q < KQ; ++q) {
                    v = FROW ? __builtin_amdgcn_raw_buffer_load_b64(rsF, in ? (int)(of[q] + 8 * (c + i)) : -1, 0, 0)
                             : __builtin_amdgcn_raw_buffer_load_b64(rsF, (int)(of[q] + i * k8), (int)(row * k8), 0);
                    x.f[q][i] = make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
                }
            }
        };
        auto compute = [&](const GradChunk<KQ> &x, int ch) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool in = ch * GR_CH + 4 * half + i < n;
                const float wx = in ? x.w1[i].x + x.w2[i].x : 0.f, wy = in ? x.w1[i].y + x.w2[i].y : 0.f;
#pragma unroll
                for (int q = 0; q < KQ; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(wx, comp ? -x.f[q][i].y : x.f[q][i].x, acc[q], 0, 0, 0);
#pragma unroll
                for (int q = 0; q < KQ; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(wy, comp ? x.f[q][i].x : x.f[q][i].y, acc[q], 0, 0, 0);
            }
        };
        const int nch = (n + GR_CH - 1) / GR_CH;
        GradChunk<KQ> x0, x1;
        int ch = wave;
        if (ch < nch) {
            load(x0, ch);
            for (; ch + 4 < nch; ch += 8) {
                load(x1, ch + 4);
                __builtin_amdgcn_sched_barrier(0);
                compute(x0, ch);
                load(x0, ch + 8);   // past the end: reads nothing or is not used
                __builtin_amdgcn_sched_barrier(0);
                compute(x1, ch + 4);
            }
            if (ch < nch) compute(x0, ch);
        }
    }

    // lane (j32, half) holds component comp of rank entry 16 q + j32 / 2 for out-rows acc_row(r, lane)
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        if (q) __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) smem[(wave * 16 + r) * GP_P + lane] = acc[q][r];
        __syncthreads();
#pragma unroll
        for (int e = t; e < 512; e += 256) {   // entries of the block, in the order of the output
            const int row = colside ? e & 31 : e >> 4, n = colside ? e >> 5 : e & 15;
            const int o = ((row & 3) + 4 * (row >> 3)) * GP_P + 32 * ((row >> 2) & 1) + 2 * n;
            float2 s = *reinterpret_cast<const float2 *>(smem + o);
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const float2 v = *reinterpret_cast<const float2 *>(smem + w * 16 * GP_P + o);
                s.x += v.x;
                s.y += v.y;
            }
            if (row < nout && 16 * q + n < kn) {
                if (colside) g[td.offB + (int64_t)(b0 + 16 * q + n) * td.dj + a0 + row] = s;   // G_R^T
                else g[td.offA + (int64_t)(a0 + row) * k + b0 + 16 * q + n] = s;
            }
        }
    }
}

__global__ __launch_bounds__(256, 2) void grad_kernel(const TileDesc *__restrict__ tiles,
                                                   const GradItem *__restrict__ items,
                                                   const ProbOff *__restrict__ probs,
                                                   const float2 *__restrict__ W_base,
                                                   const float2 *__restrict__ theta_base,
                                                   float2 *__restrict__ g_base) {
    constexpr int SM_G = 4 * 16 * GP_P;
    constexpr int SM_Z = 2 * GZ_BC * (GZ_BR + 1);
    __shared__ __attribute__((aligned(8))) float smem[SM_G > SM_Z ? SM_G : SM_Z];
    const GradItem it = items[blockIdx.x];
    const TileDesc td = tiles[it.tile];
    const ProbOff po = probs[it.prob];
    const float2 *W = W_base + po.x;
    const int64_t ldw = po.ldx;
    const float2 *theta = theta_base + po.theta;
    float2 *g = g_base + po.theta;
    const int t = threadIdx.x;

    if (it.kind == G_Z) {
        // grad Z = (W_ii + W_ii^T)/2 on the block rows a0.., cols b0..
        float2 *sW = reinterpret_cast<float2 *>(smem);
        const int d = td.di;
        const int a0 = it.a0, b0 = it.b0;
        const int nrow = min(GZ_BR, d - a0), ncol = min(GZ_BC, d - b0);
        for (int e = t; e < GZ_BC * GZ_BR; e += 256) {
            const int cc = e >> 5, rr = e & 31;
            float2 v = make_float2(0.f, 0.f);
            if (cc < ncol && rr < nrow) v = W[(td.row0 + b0 + cc) * ldw + td.col0 + a0 + rr];
            sW[cc * (GZ_BR + 1) + rr] = v;
        }
        __syncthreads();
        for (int e = t; e < GZ_BR * GZ_BC; e += 256) {
            const int rr = e >> 6, cc = e & 63;
            if (rr < nrow && cc < ncol) {
                const float2 wd = W[(td.row0 + a0 + rr) * ldw + td.col0 + b0 + cc];
                const float2 wt = sW[cc * (GZ_BR + 1) + rr];
                g[td.offA + (int64_t)(a0 + rr) * d + b0 + cc] =
                    make_float2(0.5f * (wd.x + wt.x), 0.5f * (wd.y + wt.y));
            }
        }
        return;
    }
    auto go = [&](auto kq) {
        if (it.kind == G_L) grad_block<decltype(kq)::value, true>(it, td, W, ldw, theta, g, smem);
        else grad_block<decltype(kq)::value, false>(it, td, W, ldw, theta, g, smem);
    };
    switch (it.kq) {
        case 1: go(std::integral_constant<int, 1>()); break;
        case 2: go(std::integral_constant<int, 2>()); break;
        case 3: go(std::integral_constant<int, 3>()); break;
        default: go(std::integral_constant<int, 4>()); break;
    }
}

}  // namespace

hipError_t launch_assemble(bool dir, const TileDesc *tiles, const AsmItem *items, int nitems,
                           const ProbOff *probs, const float2 *theta, const float2 *p,
                           float2 *X, float2 *X2, hipStream_t s, bool out_bf16, int64_t x2_words,
                           int64_t lo_words) {
    if (nitems <= 0) return hipSuccess;
    const dim3 g(nitems), b(256);
    if (dir && out_bf16)
        hipLaunchKernelGGL((assemble_kernel<true, true>), g, b, 0, s, tiles, items, probs, theta, p, X, X2, x2_words, lo_words);
    else if (dir)
        hipLaunchKernelGGL((assemble_kernel<true, false>), g, b, 0, s, tiles, items, probs, theta, p, X, X2, x2_words, lo_words);
    else if (out_bf16)
        hipLaunchKernelGGL((assemble_kernel<false, true>), g, b, 0, s, tiles, items, probs, theta, p, X, X2, x2_words, lo_words);
    else
        hipLaunchKernelGGL((assemble_kernel<false, false>), g, b, 0, s, tiles, items, probs, theta, p, X, X2, x2_words, lo_words);
    return hipGetLastError();
}

hipError_t launch_grad(const TileDesc *tiles, const GradItem *items, int nitems,
                       const ProbOff *probs, const float2 *W, const float2 *theta, float2 *g,
                       hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(grad_kernel, dim3(nitems), dim3(256), 0, s, tiles, items, probs, W, theta, g);
    return hipGetLastError();
}

}  // namespace tlr
