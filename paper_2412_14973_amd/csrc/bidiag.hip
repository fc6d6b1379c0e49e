// Singular-value counts of the tiles in FP64 for the rank / tile-size estimate (Hyper-parameter selection and
// initialization; the examples' rank study): k = #{sigma >= eps v0} per tile, without the singular vectors.
//
// Every tile is reduced to a real bidiagonal B by Householder reflections (Golub-Kahan, |d_i| and |e_i| only,
// which is all that its singular values depend on), and singular values are counted on B by the signs of the
// stationary quotient-difference recurrence of B^T B - t^2 (Fernando and Parlett's form of Sturm's count).
// v0 comes from the same count by repeated subdivision of the interval that holds the largest one. All of it is
// backward stable in FP64: a count is exact for singular values further than a few n 1e-16 v0 from t.
//
// One workgroup per tile. Step k: the reflection u of column k; all columns c > k take the right reflection
// of step k - 1, A -= zt v^H, and the left one, A -= conj(tau) u (u^H A), in one pass (32 lanes per column, its
// rows in registers); the reflection v of row k; zt = tau A v in a second, reading pass. What bounds it is the
// latency of a step's five phases: about 5 us a step with the tile in registers (up to 128 rows, and the last 128
// rows of tiles up to 256) and 24 to 26 with it in memory (the first steps of a 256-row tile: through one CU, two
// reads and one write of the rest of the tile; half the bytes gave 7 %). Tiles up to 32 rows in a launch of their
// own are held in LDS. Tile sizes 64, 128 and 256 of a 1024 x 1024 matrix, in one launch: 4.0 ms (6.0 with a launch
// each and all steps in memory), where one-sided Jacobi with a launch per round of rotations took 48.6 ms (6104
// launches of 8 us).
#include "svd.hpp"

#include "common.hpp"

namespace tlr {
namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 fma_c(double2 a, double2 b, double2 c) {   // a b + c
    return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 conj_c(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 neg_c(double2 a) { return make_double2(-a.x, -a.y); }

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// sum over the 16 lanes of a DPP row, in every lane: pairs, quads, halves, the row (a fixed order)
__device__ __forceinline__ double sum16(double v) {
    v += dpp<0xB1>(v);    // quad_perm 1 0 3 2
    v += dpp<0x4E>(v);    // quad_perm 2 3 0 1
    v += dpp<0x141>(v);   // row_half_mirror
    v += dpp<0x140>(v);   // row_mirror
    return v;
}
// the other half's value of a pair of rows of 16 lanes, and of the wave's two halves of 32
__device__ __forceinline__ double swap16(double v) {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    const bool odd = threadIdx.x & 16;
    return __longlong_as_double(((long long)(odd ? hi[0] : hi[1]) << 32) | (odd ? lo[0] : lo[1]));
}
__device__ __forceinline__ double sum32(double v) {
    v = sum16(v);
    return v + swap16(v);
}
__device__ __forceinline__ double sum64(double v) {
    v = sum32(v);
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    const bool up = threadIdx.x & 32;
    return v + __longlong_as_double(((long long)(up ? hi[0] : hi[1]) << 32) | (up ? lo[0] : lo[1]));
}
// lane l's value (l uniform)
__device__ __forceinline__ double of_lane(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | lo);
}

__device__ __forceinline__ double recip(double p) {   // two Newton steps on the hardware's estimate
    double r = __builtin_amdgcn_rcp(p);
    r = fma(fma(-p, r, 1.0), r, r);
    return fma(fma(-p, r, 1.0), r, r);
}
__device__ __forceinline__ double root(double x) {   // likewise
    double r = __builtin_amdgcn_rsq(x);
    r = fma(fma(-x * r, r, 1.0), 0.5 * r, r);
    r = fma(fma(-x * r, r, 1.0), 0.5 * r, r);
    const double s = x * r;
    return fma(fma(-s, s, x), 0.5 * r, s);
}

// reflection I - tau v v^H (v_0 = 1) that takes (alpha, x) to (beta, 0), beta real; none where all of it is zero or
// its squares underflow (the entries are FP32 numbers)
struct Reflect {
    double beta;
    double2 tau, scale;   // v = scale x below alpha
};
__device__ __forceinline__ Reflect reflect(double2 alpha, double xnorm2) {
    Reflect h;
    const double y2 = fma(alpha.y, alpha.y, xnorm2), n2 = fma(alpha.x, alpha.x, y2);
    if (y2 == 0.0 || n2 < 1e-280) {
        h.beta = alpha.x;
        h.tau = h.scale = make_double2(0.0, 0.0);
        return h;
    }
    const double nrm = root(n2);
    h.beta = alpha.x >= 0.0 ? -nrm : nrm;
    const double rb = recip(h.beta);
    const double2 d = make_double2(alpha.x - h.beta, alpha.y);
    h.tau = make_double2(-d.x * rb, -alpha.y * rb);
    const double q = recip(fma(d.x, d.x, d.y * d.y));
    h.scale = make_double2(d.x * q, -d.y * q);
    return h;
}

// how many singular values of the bidiagonal are >= t (d2, e2: squares, scaled with t so that the largest is of
// the order of 1: no step over- or underflows; nor do a t far above all of them, which needs no count, and one whose
// square vanishes, which only an exact zero is below)
__device__ __forceinline__ int at_least(const double *d2, const double *e2, int n, double t) {
    if (!(t > 0.0)) return n;
    if (t >= 4.0) return 0;
    const double t2 = fmax(t * t, 2.3e-308);
    double s = -t2;
    int below = 0;
    for (int i = 0; i < n; ++i) {
        double p = d2[i] + s;
        below += p < 0.0 ? 1 : 0;
        if (fabs(p) < 1e-200) p = p < 0.0 ? -1e-200 : 1e-200;
        s = fma(s, e2[i] * recip(p), -t2);   // e2[n - 1] = 0
    }
    return n - below;
}
// the power of two that brings v to [1/2, 1)
__device__ __forceinline__ double scale_of(double v) { return v > 0.0 ? ldexp(1.0, -ilogb(v) - 1) : 1.0; }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// A tile in L2 through buffer instructions: an offset past its end reads zero and writes nothing, so every
// access of a pass is unconditional and they are all in flight together.
struct TileMem {
    __amdgpu_buffer_rsrc_t rs;
    __device__ double2 get(uint32_t off) const {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
        return make_double2(__hiloint2double(v.y, v.x), __hiloint2double(v.w, v.z));
    }
    __device__ void put(uint32_t off, double2 x) const {
        const u32x4 v = {(unsigned)__double2loint(x.x), (unsigned)__double2hiint(x.x), (unsigned)__double2loint(x.y),
                         (unsigned)__double2hiint(x.y)};
        __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)off, 0, 0);
    }
};
// a tile in LDS, the same offsets
struct TileLds {
    double2 *a;
    __device__ double2 get(uint32_t off) const { return a[min(off >> 4, last)]; }
    __device__ void put(uint32_t off, double2 x) const {
        if ((off >> 4) < last) a[off >> 4] = x;
    }
    uint32_t last;   // entries; a[last] is zero
};
constexpr uint32_t OUTSIDE = 0xfffffff0u;

// What a workgroup keeps in LDS besides the tile (or the share of it): the vectors of the step, zero past row m.
template <int MMAX, int NT>
struct Shared {
    double2 part[NT / 64 * MMAX];
    double2 su[MMAX], szt[MMAX], sv[MMAX], srow[MMAX], scol[MMAX];
    double sd2[MMAX], se2[MMAX];
    double2 stau;
    int sbest;
};

// The steps' phases, with barriers between them. m x n: the tile, m >= n; MMAX >= m.
template <int MMAX, int NT>
struct Steps {
    static constexpr int NW = NT / 64, NG = NT / 32;   // waves; groups of 32 lanes
    static constexpr int MR = MMAX / 32;               // rows per lane of a group
    static constexpr int ML = (MMAX + 63) / 64;        // rows per lane of a wave
    double2 *part, *su, *szt, *sv, *srow, *scol;       // part: [NW][MMAX]
    double *sd2, *se2;
    double2 *stau;
    int *sbest;
    int m, n;

    template <int MS>
    __device__ Steps(Shared<MS, NT> &s, int m_, int n_)
        : part(s.part), su(s.su), szt(s.szt), sv(s.sv), srow(s.srow), scol(s.scol), sd2(s.sd2), se2(s.se2), stau(&s.stau),
          sbest(&s.sbest), m(m_), n(n_) {
        static_assert(MS >= MMAX, "the buffers hold the tile");
    }

    __device__ void clear() const {
        for (int r = threadIdx.x; r < MMAX; r += NT) {
            su[r] = szt[r] = sv[r] = srow[r] = scol[r] = make_double2(0.0, 0.0);
            sd2[r] = se2[r] = 0.0;
        }
    }

    // column k (scol: after the left reflections so far, without the last right one), by one wave
    __device__ void column(int k) const {
        const int lane = threadIdx.x & 63;
        const double2 cv = conj_c(sv[k]);
        double2 x[ML];
        double nn = 0.0;
#pragma unroll
        for (int i = 0; i < ML; ++i) {
            const int r = lane + 64 * i;
            x[i] = make_double2(0.0, 0.0);
            if (r >= k && r < m) {
                x[i] = fma_c(neg_c(szt[r]), cv, scol[r]);
                if (r > k) nn = fma(x[i].x, x[i].x, fma(x[i].y, x[i].y, nn));
            }
        }
        nn = sum64(nn);
        double2 alpha = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < ML; ++i)
            if (k >> 6 == i) alpha = make_double2(of_lane(x[i].x, k & 63), of_lane(x[i].y, k & 63));
        const Reflect h = reflect(alpha, nn);
#pragma unroll
        for (int i = 0; i < ML; ++i) {
            const int r = lane + 64 * i;
            // zero above the diagonal: the passes below need no test of their rows against k
            if (r < m) su[r] = r < k ? make_double2(0.0, 0.0) : r == k ? make_double2(1.0, 0.0) : cmul(x[i], h.scale);
        }
        if (lane == 0) {
            sd2[k] = h.beta * h.beta;
            *stau = conj_c(h.tau);
        }
    }

    // row k, columns > k: its reflection from the right, by one wave
    __device__ void row(int k) const {
        const int lane = threadIdx.x & 63;
        double2 x[ML];
        double nn = 0.0;
#pragma unroll
        for (int i = 0; i < ML; ++i) {
            const int c = lane + 64 * i;
            x[i] = make_double2(0.0, 0.0);
            if (c > k && c < n) {
                x[i] = conj_c(srow[c]);
                if (c > k + 1) nn = fma(x[i].x, x[i].x, fma(x[i].y, x[i].y, nn));
            }
        }
        nn = sum64(nn);
        const int k1 = k + 1;
        double2 alpha = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < ML; ++i)
            if (k1 >> 6 == i) alpha = make_double2(of_lane(x[i].x, k1 & 63), of_lane(x[i].y, k1 & 63));
        const Reflect h = reflect(alpha, nn);
#pragma unroll
        for (int i = 0; i < ML; ++i) {
            const int c = lane + 64 * i;
            if (c > k && c < n) sv[c] = c == k1 ? make_double2(1.0, 0.0) : cmul(x[i], h.scale);
        }
        if (lane == 0) {
            se2[k] = h.beta * h.beta;
            *stau = h.tau;
        }
    }

    // columns c > k of a tile in memory: the right reflection of step k - 1 and the left one of step k
    template <class MEM>
    __device__ void left(const MEM &mem, int k) const {
        const int l32 = threadIdx.x & 31, grp = threadIdx.x >> 5;
        const double2 tau = *stau;
        double2 u[MR], zt[MR];   // of this lane's rows, the same for all columns
#pragma unroll
        for (int j = 0; j < MR; ++j) {
            u[j] = su[l32 + 32 * j];
            zt[j] = neg_c(szt[l32 + 32 * j]);
        }
        // rows of 32 that lie above row k, and rows past m, are left out
        auto off = [&](int c, int j) {
            return 32 * j + 31 >= k && l32 + 32 * j < m && c < n ? 16u * (uint32_t)(c * m + l32) + 512u * j : OUTSIDE;
        };
        auto load = [&](double2 (&a)[MR], int c) {
#pragma unroll
            for (int j = 0; j < MR; ++j) a[j] = mem.get(off(c, j));
        };
        auto update = [&](double2 (&a)[MR], int c) {
            const double2 cv = conj_c(sv[c]);
            double yr = 0.0, yi = 0.0;
#pragma unroll
            for (int j = 0; j < MR; ++j)
                if (32 * j + 31 >= k) {   // uniform
                    a[j] = fma_c(zt[j], cv, a[j]);
                    yr = fma(u[j].x, a[j].x, fma(u[j].y, a[j].y, yr));   // conj(u) a
                    yi = fma(u[j].x, a[j].y, fma(-u[j].y, a[j].x, yi));
                }
            const double2 y = neg_c(cmul(tau, make_double2(sum32(yr), sum32(yi))));
#pragma unroll
            for (int j = 0; j < MR; ++j) {
                a[j] = fma_c(u[j], y, a[j]);
                mem.put(off(c, j), a[j]);
            }
#pragma unroll
            for (int j = 0; j < MR; ++j) {
                const int r = l32 + 32 * j;
                if (r == k) srow[c] = a[j];
                if (c == k + 1 && r < m) scol[r] = a[j];
            }
        };
        double2 a[MR];
        if constexpr (MR <= 8) {   // the next column's loads ahead of a column's work, where the registers hold both
            double2 b[MR];
            int c = k + 1 + grp;
            load(a, c);
            for (; c < n; c += 2 * NG) {
                load(b, c + NG);
                update(a, c);
                if (c + NG >= n) break;
                load(a, c + 2 * NG);
                update(b, c + NG);
            }
        } else {
            for (int c = k + 1 + grp; c < n; c += NG) {
                load(a, c);
                update(a, c);
            }
        }
    }

    // the waves' parts of zt = A v over the rows > k of a tile in memory
    template <class MEM>
    __device__ void right(const MEM &mem, int k) const {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        double2 z[ML];
#pragma unroll
        for (int i = 0; i < ML; ++i) z[i] = make_double2(0.0, 0.0);
        constexpr int CC = ML <= 4 ? 32 / NW : 1;   // columns in flight
        for (int c0 = k + 1 + wave; c0 < n; c0 += CC * NW) {
            double2 a[CC][ML];
#pragma unroll
            for (int q = 0; q < CC; ++q) {
                const int c = c0 + q * NW;
#pragma unroll
                for (int i = 0; i < ML; ++i) {
                    const int r = lane + 64 * i;
                    a[q][i] = mem.get(64 * i + 63 > k && r < m && c < n ? 16u * (uint32_t)(c * m + r) : OUTSIDE);
                }
            }
#pragma unroll
            for (int q = 0; q < CC; ++q) {
                const double2 v = sv[min(c0 + q * NW, n - 1)];
#pragma unroll
                for (int i = 0; i < ML; ++i) z[i] = fma_c(a[q][i], v, z[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < ML; ++i) {
            const int r = lane + 64 * i;
            if (r < m) part[wave * MMAX + r] = z[i];
        }
    }
    __device__ void add_parts(int k) const {
        for (int r = threadIdx.x; r < m; r += NT) {
            double2 z = part[r];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                z.x += part[w * MMAX + r].x;
                z.y += part[w * MMAX + r].y;
            }
            szt[r] = r > k ? cmul(*stau, z) : make_double2(0.0, 0.0);
        }
    }

    // steps k0 .. k1 - 1 of a tile in memory (all of a step but the last column's, which has no row)
    template <class MEM>
    __device__ void in_memory(const MEM &mem, int k0, int k1) const {
        const int wave = threadIdx.x >> 6;
        for (int k = k0; k < k1; ++k) {
            if (wave == 0) column(k);
            if (k == n - 1) break;
            __syncthreads();
            left(mem, k);
            __syncthreads();
            if (wave == 0) row(k);
            __syncthreads();
            right(mem, k);
            __syncthreads();
            add_parts(k);
            __syncthreads();
        }
        __syncthreads();
    }

    // Steps k0 .. n - 1 with the rest of the tile, at most RB x RB, in registers: lane l32 of group grp holds rows
    // k0 + l32 + 32 j of columns k0 + grp + NG q. load(r, c) gives the tile's entries.
    template <int RB, class F>
    __device__ void in_registers(int k0, F &&load) const {
        constexpr int QR = RB / 32, QC = RB / NG;
        static_assert(NG % 4 == 0 && 4 * RB <= NT, "four threads add a row's parts");
        const int l32 = threadIdx.x & 31, grp = threadIdx.x >> 5, wave = threadIdx.x >> 6;
        double2 a[QC][QR];   // [column][row]
#pragma unroll
        for (int q = 0; q < QC; ++q)
#pragma unroll
            for (int j = 0; j < QR; ++j) {
                const int r = k0 + l32 + 32 * j, c = k0 + grp + NG * q;
                a[q][j] = r < m && c < n ? load(r, c) : make_double2(0.0, 0.0);
            }
        if (k0 == 0 && grp == 0)
#pragma unroll
            for (int j = 0; j < QR; ++j) scol[l32 + 32 * j] = a[0][j];
        __syncthreads();
        for (int k = k0; k < n; ++k) {
            if (wave == 0) column(k);
            if (k == n - 1) break;
            __syncthreads();
            const int kl = k - k0;
            {
                const double2 tau = *stau;
                double2 u[QR], zt[QR];
#pragma unroll
                for (int j = 0; j < QR; ++j) {
                    u[j] = su[k0 + l32 + 32 * j];
                    zt[j] = neg_c(szt[k0 + l32 + 32 * j]);
                }
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int c = k0 + grp + NG * q;
                    if (c <= k || c >= n) continue;   // the same for a group's lanes
                    const double2 cv = conj_c(sv[c]);
                    double yr = 0.0, yi = 0.0;
#pragma unroll
                    for (int j = 0; j < QR; ++j)
                        if (32 * j + 31 >= kl) {   // uniform
                            a[q][j] = fma_c(zt[j], cv, a[q][j]);
                            yr = fma(u[j].x, a[q][j].x, fma(u[j].y, a[q][j].y, yr));   // conj(u) a
                            yi = fma(u[j].x, a[q][j].y, fma(-u[j].y, a[q][j].x, yi));
                        }
                    const double2 y = neg_c(cmul(tau, make_double2(sum32(yr), sum32(yi))));
#pragma unroll
                    for (int j = 0; j < QR; ++j) {
                        if (32 * j + 31 >= kl) a[q][j] = fma_c(u[j], y, a[q][j]);
                        const int r = k0 + l32 + 32 * j;
                        if (r == k) srow[c] = a[q][j];
                        if (c == k + 1) scol[r] = a[q][j];
                    }
                }
            }
            __syncthreads();
            if (wave == 0) row(k);
            __syncthreads();
            {
                double2 z[QR];
#pragma unroll
                for (int j = 0; j < QR; ++j) z[j] = make_double2(0.0, 0.0);
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int c = k0 + grp + NG * q;
                    if (c <= k || c >= n) continue;
                    const double2 v = sv[c];
#pragma unroll
                    for (int j = 0; j < QR; ++j) z[j] = fma_c(a[q][j], v, z[j]);
                }
#pragma unroll
                for (int j = 0; j < QR; ++j) part[grp * RB + l32 + 32 * j] = z[j];
            }
            __syncthreads();
            // four threads per row add a quarter of the groups each
            if (threadIdx.x < 4 * RB) {
                const int r = threadIdx.x >> 2, g0 = (threadIdx.x & 3) * (NG / 4);
                double2 z = part[g0 * RB + r];
#pragma unroll
                for (int g = 1; g < NG / 4; ++g) {
                    z.x += part[(g0 + g) * RB + r].x;
                    z.y += part[(g0 + g) * RB + r].y;
                }
                z.x += dpp<0xB1>(z.x);
                z.y += dpp<0xB1>(z.y);
                z.x += dpp<0x4E>(z.x);
                z.y += dpp<0x4E>(z.y);
                if ((threadIdx.x & 3) == 0 && k0 + r < m) szt[k0 + r] = r > kl ? cmul(*stau, z) : make_double2(0.0, 0.0);
            }
            __syncthreads();
        }
        __syncthreads();
    }

    // the largest singular value: its interval cut in NS + 1 parts until it is a rounding wide; and the squares for
    // the counts: d2 in the tile's sigma slots, e2 at the start of its W and the largest singular value behind them
    __device__ void finish(double *d2, double *e2) const {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        double lo = 0.0, hi = 0.0;
        for (int i = tid; i < n; i += NT) {
            const double d = sqrt(sd2[i]), e = sqrt(se2[i]), e0 = i ? sqrt(se2[i - 1]) : 0.0;
            lo = fmax(lo, fmax(d, e));
            hi = fmax(hi, d + fmax(e, e0));
        }
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmax(lo, __shfl_xor(lo, o, 64));
            hi = fmax(hi, __shfl_xor(hi, o, 64));
        }
        if (lane == 0) part[wave] = make_double2(lo, hi);
        __syncthreads();
        for (int w = 0; w < NW; ++w) {
            lo = fmax(lo, part[w].x);
            hi = fmax(hi, part[w].y);
        }
        hi = fmax(hi * (1.0 + 1e-14), lo);
        lo *= 1.0 - 1e-14;
        const double sc = scale_of(hi);
        // (the largest singular value lies between the largest entry and the largest row sum)
        __syncthreads();
        for (int i = tid; i < n; i += NT) {
            sd2[i] *= sc * sc;
            se2[i] *= sc * sc;
        }
        lo *= sc;
        hi *= sc;
        constexpr int NS = NT < 256 ? NT : 256;   // points per cut: one wave per SIMD, the recurrence is a serial chain
        for (int it = 0; it < 9 && hi - lo > 1e-16 * hi; ++it) {
            const double step = (hi - lo) / (NS + 1);
            if (tid == 0) *sbest = 0;
            __syncthreads();
            if (tid < NS && at_least(sd2, se2, n, fma(step, tid + 1, lo)) > 0) atomicMax(sbest, tid + 1);
            __syncthreads();
            const int b = *sbest;
            __syncthreads();
            const double nlo = fma(step, b, lo);
            hi = b == NS ? hi : fma(step, b + 1, lo);
            lo = nlo;
        }
        // the lower end: counted as reached, so that a threshold of v0 itself counts the value it comes from
        if (tid == 0) e2[n] = lo / sc;
        for (int i = tid; i < n; i += NT) {
            d2[i] = sd2[i] / (sc * sc);
            e2[i] = se2[i] / (sc * sc);
        }
    }
};

__device__ __forceinline__ TileMem tile_mem(double2 *W, const SvdTile &t) {
    return TileMem{__builtin_amdgcn_make_buffer_rsrc((void *)(W + t.offW), (short)0, t.m * t.n * 16, 0x00020000)};
}

// NT threads, tiles up to MMAX rows, all steps in memory; RES: in LDS, and read from X, else in W
template <int MMAX, int NT, bool RES>
__global__ __launch_bounds__(NT) void bidiag_kernel(const SvdTile *__restrict__ tiles, const float2 *__restrict__ X,
                                                    int64_t ldx, double2 *__restrict__ W, double *__restrict__ d2out,
                                                    int32_t *__restrict__ nonfinite) {
    __shared__ double2 sA[RES ? MMAX * MMAX + 1 : 1];
    __shared__ Shared<MMAX, NT> sh;
    const SvdTile t = tiles[blockIdx.x];
    const int m = t.m, n = t.n;
    const Steps<MMAX, NT> st(sh, m, n);
    // the tile, column-major, ld m
    const auto mem = [&] {
        if constexpr (RES) return TileLds{sA, (uint32_t)(m * n)};
        else return tile_mem(W, t);
    }();
    if (RES) {
        bool ok = true;
        for (int e = threadIdx.x; e < m * n; e += NT) {   // read along the rows of X
            const int i = t.trans ? e / m : e / n, j = t.trans ? e % m : e % n;
            const float2 x = X[(t.row0 + i) * ldx + t.col0 + j];
            ok = ok && isfinite(x.x) && isfinite(x.y);
            sA[t.trans ? i * m + j : j * m + i] = make_double2(x.x, x.y);
        }
        if (threadIdx.x == 0) sA[m * n] = make_double2(0.0, 0.0);
        if (!ok) *nonfinite = 1;
    }
    st.clear();
    __syncthreads();
    for (int r = threadIdx.x; r < m; r += NT) st.scol[r] = mem.get(16 * r);
    __syncthreads();
    st.in_memory(mem, 0, n);
    st.finish(d2out + t.offS, reinterpret_cast<double *>(W + t.offW));
}

// Tiles of up to 256 rows, of several sizes in one launch: up to 128 rows all of a tile's steps are in registers, read
// from X; above, those before the last 128 rows are in memory (W).
constexpr int REG_NT = 512;
__global__ __launch_bounds__(REG_NT) void bidiag_reg_kernel(const SvdTile *__restrict__ tiles, const float2 *__restrict__ X,
                                                          int64_t ldx, double2 *__restrict__ W,
                                                          double *__restrict__ d2out, int32_t *__restrict__ nonfinite) {
    __shared__ Shared<256, REG_NT> sh;
    const SvdTile t = tiles[blockIdx.x];
    const int m = t.m, n = t.n;
    double *d2 = d2out + t.offS, *e2 = reinterpret_cast<double *>(W + t.offW);
    bool ok = true;
    auto from_x = [&](int r, int c) {
        const float2 x = X[(t.row0 + (t.trans ? c : r)) * ldx + t.col0 + (t.trans ? r : c)];
        ok = ok && isfinite(x.x) && isfinite(x.y);
        return make_double2(x.x, x.y);
    };
    if (m <= 64) {
        const Steps<64, REG_NT> st(sh, m, n);
        st.clear();
        __syncthreads();
        st.in_registers<64>(0, from_x);
        st.finish(d2, e2);
    } else if (m <= 128) {
        const Steps<128, REG_NT> st(sh, m, n);
        st.clear();
        __syncthreads();
        st.in_registers<128>(0, from_x);
        st.finish(d2, e2);
    } else {
        const Steps<256, REG_NT> st(sh, m, n);
        const TileMem mem = tile_mem(W, t);
        const int k0 = m - 128;
        st.clear();
        __syncthreads();
        for (int r = threadIdx.x; r < m; r += REG_NT) st.scol[r] = mem.get(16 * r);
        __syncthreads();
        st.in_memory(mem, 0, min(k0, n));
        if (k0 < n) st.in_registers<128>(k0, [&](int r, int c) { return mem.get(16u * (uint32_t)(c * m + r)); });
        st.finish(d2, e2);
    }
    if (!ok) *nonfinite = 1;
}

__global__ __launch_bounds__(256) void vmax_kernel(const SvdTile *__restrict__ tiles, int ntiles,
                                                   const int32_t *__restrict__ first, const double2 *__restrict__ W,
                                                   double *__restrict__ v0) {
    __shared__ double red[256];
    const int i0 = first ? first[blockIdx.x] : 0, i1 = first ? first[blockIdx.x + 1] : ntiles;
    double x = 0.0;
    for (int i = i0 + threadIdx.x; i < i1; i += 256)
        x = fmax(x, reinterpret_cast<const double *>(W + tiles[i].offW)[tiles[i].n]);
    red[threadIdx.x] = x;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) v0[blockIdx.x] = red[0];
}

// k of every tile (one workgroup each: the squares through LDS, the recurrence in one lane)
__global__ __launch_bounds__(64) void count_kernel(const SvdTile *__restrict__ tiles, const double2 *__restrict__ W,
                                                   const double *__restrict__ d2, const double *__restrict__ v0,
                                                   double eps, int32_t *__restrict__ kout) {
    __shared__ double sd2[BIDIAG_MAX_M], se2[BIDIAG_MAX_M];
    const SvdTile t = tiles[blockIdx.x];
    const double *e2 = reinterpret_cast<const double *>(W + t.offW);
    const double v = v0[t.grid], sc = scale_of(v);
    for (int i = threadIdx.x; i < t.n; i += 64) {
        sd2[i] = d2[t.offS + i] * (sc * sc);
        se2[i] = e2[i] * (sc * sc);
    }
    __syncthreads();
    if (threadIdx.x == 0) kout[blockIdx.x] = at_least(sd2, se2, t.n, eps * v * sc);
}

}  // namespace

bool bidiag_reads_x(int mmax) { return mmax <= 128; }

bool bidiag_shared(int64_t mmax) { return mmax > 32 && mmax <= 256; }

hipError_t launch_bidiag(const SvdTile *tiles, int ntiles, bool mixed, int mmax, const float2 *X, int64_t ldx, double2 *W,
                         double *d2, int32_t *nonfinite, hipStream_t s) {
    if (ntiles <= 0) return hipSuccess;
    const dim3 g((unsigned)ntiles);
    if (mixed && mmax > 256) return hipErrorInvalidValue;
    if (mmax <= 32 && !mixed)
        hipLaunchKernelGGL((bidiag_kernel<32, 256, true>), g, dim3(256), 0, s, tiles, X, ldx, W, d2, nonfinite);
    else if (mmax <= 256)
        hipLaunchKernelGGL(bidiag_reg_kernel, g, dim3(REG_NT), 0, s, tiles, X, ldx, W, d2, nonfinite);
    else if (mmax <= BIDIAG_MAX_M)
        hipLaunchKernelGGL((bidiag_kernel<512, 512, false>), g, dim3(512), 0, s, tiles, X, ldx, W, d2, nonfinite);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_svd_counts(const SvdTile *tiles, int ntiles, const int32_t *first, int ngrids, const double2 *W,
                             const double *d2, double eps, int32_t *kout, double *v0, hipStream_t s) {
    if (ntiles <= 0) return hipSuccess;
    if (ngrids < 1 || (ngrids > 1 && !first)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(vmax_kernel, dim3((unsigned)ngrids), dim3(256), 0, s, tiles, ntiles, first, W, v0);
    hipLaunchKernelGGL(count_kernel, dim3((unsigned)ntiles), dim3(64), 0, s, tiles, W, d2, v0, eps, kout);
    return hipGetLastError();
}

}  // namespace tlr
