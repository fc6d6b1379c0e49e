// Memory-bound kernels: staging of D, column permutation (eq. axb_sd), and the
// optimiser's vector / scalar work (L-BFGS two-loop recursion, exact line
// search, updates). All reductions are FP64, deterministic (fixed-order
// per-segment partials, then one fixed-order tree per problem), with no
// atomics. Scalars never leave the device.
#include <cstddef>

#include "common.hpp"
#include "exact_step.hpp"
#include "vec.hpp"

namespace tlr {
namespace {

// ---------------------------------------------------------------------------
// staging: Ds = D, padded with zeros to lds x ldk (32 x 32 entries per workgroup)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void stage_d_kernel(const float2 *__restrict__ D, int64_t ns, int64_t nr,
                                                      float2 *__restrict__ Ds, int64_t ldk, int64_t lds) {
    const int64_t s0 = (int64_t)blockIdx.y * 32, c = (int64_t)blockIdx.x * 32 + (threadIdx.x & 31);
    for (int r = threadIdx.x >> 5; r < 32; r += 8) {
        const int64_t s = s0 + r;
        if (s < lds && c < ldk) Ds[s * ldk + c] = s < ns && c < nr ? D[s * nr + c] : make_float2(0.f, 0.f);
    }
}

// a 32 x 32 block of split planes: 4 KB in a row, 16 bytes per thread
template <class F>
__device__ __forceinline__ void put_plane_block(uint32_t *hi, uint32_t *lo, int64_t base, F &&at) {
    const int t = threadIdx.x;
    const int row = t & 31, k = PLANE_KB * (t >> 6) + ((t & 32) >> 3);
    uint4 h, l;
    split_c(at(row, k), h.x, l.x);
    split_c(at(row, k + 1), h.y, l.y);
    split_c(at(row, k + 2), h.z, l.z);
    split_c(at(row, k + 3), h.w, l.w);
    reinterpret_cast<uint4 *>(hi + base)[t] = h;
    reinterpret_cast<uint4 *>(lo + base)[t] = l;
}

__global__ __launch_bounds__(256) void stage_d_split_kernel(Problems in, int64_t ns, int64_t nr,
                                                            uint32_t *__restrict__ Dh, uint32_t *__restrict__ Dl,
                                                            int64_t ldk, uint32_t *__restrict__ DHh,
                                                            uint32_t *__restrict__ DHl, int64_t lds, int64_t stride) {
    __shared__ float2 tile[32][33];
    const float2 *__restrict__ D = in.D[blockIdx.z];
    if (Dh) {
        Dh += blockIdx.z * stride;
        Dl += blockIdx.z * stride;
    }
    if (DHh) {
        DHh += blockIdx.z * stride;
        DHl += blockIdx.z * stride;
    }
    const int64_t s0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int r = ty; r < 32; r += 8) {
        const int64_t s = s0 + r, c = c0 + tx;
        float2 v = make_float2(0.f, 0.f);
        if (s < ns && c < nr) v = D[s * nr + c];
        tile[r][tx] = v;
    }
    __syncthreads();
    if (Dh) put_plane_block(Dh, Dl, plane_word(s0, c0, ldk), [&](int row, int k) { return tile[row][k]; });
    if (DHh)
        put_plane_block(DHh, DHl, plane_word(c0, s0, lds),
                        [&](int row, int k) { return make_float2(tile[k][row].x, -tile[k][row].y); });
}

// The inputs of a solve, all problems in one launch (per problem copies left a batch of small ones waiting for their
// launches: 24 launches and 16 copies for 8 problems of nr 64, a quarter of a
// five-iteration solve): padded D and U, theta, and the initial scalars. blockIdx.y is the
// problem; blockIdx.x takes STG_ROWS rows of D (unless Ds is null), then of U (unless Us is null), then 1024 entries of
// theta.
constexpr int STG_ROWS = 4;
__global__ __launch_bounds__(256) void stage_problems_kernel(Problems in, int64_t ns, int64_t nr, int64_t lds,
                                                             int64_t ldk, float2 *__restrict__ Ds,
                                                             float2 *__restrict__ Us, const ProbOff *__restrict__ probs,
                                                             float2 *__restrict__ th, SolveScalars *__restrict__ sc) {
    const int p = blockIdx.y, t = threadIdx.x;
    const int nb = (int)(lds / STG_ROWS);
    int b = blockIdx.x;
    const float2 *src = nullptr;
    float2 *dst = nullptr;
    if (Ds) {
        if (b < nb) { src = in.D[p]; dst = Ds; }
        b -= nb;
    }
    if (!src && Us) {
        if (b < nb) { src = in.U[p]; dst = Us; }
        b -= nb;
    }
    if (src) {
        const int64_t r0 = (int64_t)(b + nb) * STG_ROWS;
        dst += p * lds * ldk;
        for (int64_t c = t; c < ldk; c += 256) {
            float2 v[STG_ROWS];
#pragma unroll
            for (int r = 0; r < STG_ROWS; ++r)
                v[r] = (r0 + r < ns && c < nr) ? src[(r0 + r) * nr + c] : make_float2(0.f, 0.f);
#pragma unroll
            for (int r = 0; r < STG_ROWS; ++r) dst[(r0 + r) * ldk + c] = v[r];
        }
        return;
    }
    const int64_t n = in.theta_n[p];
    float2 *o = th + probs[p].theta;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = (int64_t)b * 1024 + 256 * u + t;
        if (i < n) o[i] = in.theta[p][i];
    }
    if (b == 0 && t == 0) {
        SolveScalars &s = sc[p];
        s.head = 0; s.count = 0; s.restart = 0; s.frozen = 0; s.gamma = 1.0; s.step = 0.0;
        s.f = 0.0; s.fdata = 0.0; s.thnorm2 = 0.0; s.tp = 0.0; s.pnorm2 = 0.0;
    }
}

// theta back to the callers' vectors
__global__ __launch_bounds__(256) void collect_theta_kernel(Problems out, const ProbOff *__restrict__ probs,
                                                            const float2 *__restrict__ th) {
    const int p = blockIdx.y;
    const int64_t n = out.theta_n[p];
    const float2 *v = th + probs[p].theta;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = (int64_t)blockIdx.x * 1024 + 256 * u + threadIdx.x;
        if (i < n) out.theta[p][i] = v[i];
    }
}

__global__ __launch_bounds__(256) void split_transpose_kernel(const float2 *__restrict__ r, int64_t ldr, int64_t rows,
                                                              int64_t cols, uint32_t *__restrict__ th, uint32_t *__restrict__ tl,
                                                              int64_t ldt, int64_t s_r, int64_t s_t) {
    __shared__ float2 tile[32][33];
    const int z = blockIdx.z;
    r += z * s_r;
    th += z * s_t;
    tl += z * s_t;
    const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int q = ty; q < 32; q += 8) {
        const int64_t i = r0 + q, j = c0 + tx;
        tile[q][tx] = (i < rows && j < cols) ? r[i * ldr + j] : make_float2(0.f, 0.f);
    }
    __syncthreads();
    put_plane_block(th, tl, plane_word(c0, r0, ldt), [&](int row, int k) { return tile[k][row]; });
}

// zero the padding (rows >= n, and columns >= n of rows < n) of ld x ld split planes
__global__ void zero_pad_kernel(uint32_t *__restrict__ base, int64_t ld, int64_t n, int64_t plane_stride,
                                int64_t batch_stride) {
    const int64_t row = blockIdx.x;
    uint32_t *p = base + (int64_t)blockIdx.z * batch_stride + (int64_t)blockIdx.y * plane_stride;
    const int64_t c0 = row < n ? n : 0;
    for (int64_t c = c0 + threadIdx.x; c < ld; c += blockDim.x) p[plane_word(row, c, ld)] = 0u;
}

__global__ void copy2d_kernel(const float2 *__restrict__ src, int64_t lds, float2 *__restrict__ dst,
                              int64_t ldd, int64_t rows, int64_t cols) {
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y)
        for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cols; c += (int64_t)gridDim.x * blockDim.x)
            dst[r * ldd + c] = src[r * lds + c];
}

// out[r, c] = in[r, perm[c]]; a perm entry outside [0, cols) gives a zero column and sets *bad
__global__ void permute_kernel(const float2 *__restrict__ in, const int64_t *__restrict__ perm,
                               float2 *__restrict__ out, int64_t rows, int64_t cols, int32_t *__restrict__ bad) {
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cols; c += (int64_t)gridDim.x * blockDim.x) {
        const int64_t q = perm[c];
        const bool ok = q >= 0 && q < cols;
        if (!ok && bad && blockIdx.y == 0) *bad = 1;
        for (int64_t r = blockIdx.y; r < rows; r += gridDim.y)
            out[r * cols + c] = ok ? in[r * cols + q] : make_float2(0.f, 0.f);
    }
}

// zero `words` 32-bit words at p (16-byte stores over the aligned body)
__global__ void fill_zero_kernel(uint32_t *__restrict__ p, int64_t words) {
    const int64_t mis = (int64_t)((16 - ((uintptr_t)p & 15)) & 15) / 4;   // words before a 16-byte boundary
    const int64_t lead = mis < words ? mis : words;
    const int64_t nvec = (words - lead) / 4;
    uint4 *v = reinterpret_cast<uint4 *>(p + lead);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t; i < nvec; i += stride) v[i] = make_uint4(0u, 0u, 0u, 0u);
    if (t < lead) p[t] = 0u;
    const int64_t tail = lead + 4 * nvec;
    if (t < words - tail) p[tail + t] = 0u;
}

// ---------------------------------------------------------------------------
// segment helpers
// ---------------------------------------------------------------------------
}  // namespace
// wave-wide FP64 sum of the ROCm device library (DPP row shifts and lane reads, fixed order, no LDS)
extern "C" __device__ double __ockl_wfred_add_f64(double);
namespace {

__device__ __forceinline__ double wave_sum64(double v) { return __ockl_wfred_add_f64(v); }

__device__ __forceinline__ int ring_slot(const SolveScalars &sc, int i, int m1) {
    int s = sc.head - 1 - i;
    s %= m1;
    if (s < 0) s += m1;
    return s;
}

// A thread's share of a segment: float4 chunks t, t + 256, t + 512, t + 768 (VEC_CH = 4096 floats).
// Segment offsets are multiples of 4 floats and lengths are even (complex entries); a problem's
// theta span is padded to an even number of complex entries, so the float4 that holds a segment's
// ragged end lies inside the span. Loads and stores are buffer instructions over the segment
// rounded up to whole float4s: chunks past the end read 0 and are not written (no branches, all
// loads of a thread in flight together); the two floats past an odd end are read as 0 and written
// back as the kernel's result for 0 inputs, inside the padding.
constexpr int VQ = VEC_CH / 1024;
struct V16 { float v[4 * VQ]; };

typedef unsigned int vu32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t seg_rsrc(const float *base, const VecSeg &sg) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)(base + sg.off), (short)0, ((sg.n + 3) & ~3) * 4, 0x00020000);
}

__device__ __forceinline__ V16 ld16(const float *__restrict__ base, const VecSeg &sg) {
    const __amdgpu_buffer_rsrc_t rs = seg_rsrc(base, sg);
    V16 r;
#pragma unroll
    for (int q = 0; q < VQ; ++q) {
        const int e = (threadIdx.x + 256 * q) * 4;
        const vu32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rs, e * 4, 0, 0);
        const bool full = e + 4 <= sg.n;   // else at most the first two floats are in the segment
        r.v[4 * q] = __uint_as_float(x.x);
        r.v[4 * q + 1] = __uint_as_float(x.y);
        r.v[4 * q + 2] = full ? __uint_as_float(x.z) : 0.f;
        r.v[4 * q + 3] = full ? __uint_as_float(x.w) : 0.f;
    }
    return r;
}

__device__ __forceinline__ void st16(float *__restrict__ base, const VecSeg &sg, const V16 &r) {
    const __amdgpu_buffer_rsrc_t rs = seg_rsrc(base, sg);
#pragma unroll
    for (int q = 0; q < VQ; ++q) {
        const int e = (threadIdx.x + 256 * q) * 4;
        const vu32x4 x = {__float_as_uint(r.v[4 * q]), __float_as_uint(r.v[4 * q + 1]),
                          __float_as_uint(r.v[4 * q + 2]), __float_as_uint(r.v[4 * q + 3])};
        __builtin_amdgcn_raw_buffer_store_b128(x, rs, e * 4, 0, 0);
    }
}

__device__ __forceinline__ double dot16(const V16 &x, const V16 &y) {
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < 4 * VQ; ++u) a = fma((double)x.v[u], (double)y.v[u], a);
    return a;
}

// N sums over a block of four waves at once, in a fixed order (thread 0 gets the totals)
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double *red) {
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = wave_sum64(v[k]);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) red[4 * k + w] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = ((red[4 * k] + red[4 * k + 1]) + red[4 * k + 2]) + red[4 * k + 3];
    __syncthreads();
}

// Gram pass of the vector-free L-BFGS direction. With h = head (the slot of the newest step s_h,
// written by the previous update): y_h = g - g_prev into Y[h]; then the real inner products of the
// new vectors (s_h, y_h, g) with every stored one. Partials per segment, 6 per ring slot j:
//   j == h : <s_h,s_h> <s_h,y_h> <y_h,y_h> <g,s_h> <g,y_h> <g,g>
//   j valid: <s_j,s_h> <s_j,y_h> <s_j,g>   <y_j,s_h> <y_j,y_h> <y_j,g>
//   else   : zeros
__global__ __launch_bounds__(256, 3) void gram_kernel(const VecSeg *__restrict__ segs, int m1,
                                                   const float *__restrict__ g, const float *__restrict__ gprev,
                                                   float *__restrict__ Yb, const float *__restrict__ Sb,
                                                   int64_t stride2, const SolveScalars *__restrict__ sc,
                                                   double *__restrict__ part) {
    __shared__ double red[6 * (MAX_LBFGS_M + 1)][4];
    const VecSeg sg = segs[blockIdx.x];
    const SolveScalars &s = sc[sg.prob];
    const int h = s.head, count = s.count;
    double *pp = part + (int64_t)sg.part * 6 * m1;
    const V16 vg = ld16(g, sg);
    const V16 vs = ld16(Sb + h * stride2, sg);
    V16 vy = ld16(gprev, sg);
    // the first held pair is loaded with the new vectors (an empty range when there is none)
    VecSeg sg0 = sg;
    if (count == 0) sg0.n = 0;
    const int j0 = ring_slot(s, 0, m1);
    V16 sj = ld16(Sb + j0 * stride2, sg0);
    V16 yj = ld16(Yb + j0 * stride2, sg0);
#pragma unroll
    for (int u = 0; u < 4 * VQ; ++u) vy.v[u] = vg.v[u] - vy.v[u];
    st16(Yb + h * stride2, sg, vy);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto wave_sums = [&](int j, double (&a)[6]) {
#pragma unroll
        for (int k = 0; k < 6; ++k) a[k] = wave_sum64(a[k]);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int k = 0; k < 6; ++k) red[6 * j + k][wave] = a[k];
    };
    {
        double a[6] = {dot16(vs, vs), dot16(vs, vy), dot16(vy, vy), dot16(vg, vs), dot16(vg, vy), dot16(vg, vg)};
        wave_sums(h, a);
    }
    // the held pairs, each one's loads issued before the sums of the previous one; the waves' sums are added at the
    // end, so no wave waits for another on the way
    for (int i = 0; i < count; ++i) {
        const int j = ring_slot(s, i, m1);
        VecSeg sgn = sg;   // past the last pair: an empty range, the loads return 0 and move no data
        if (i + 1 >= count) sgn.n = 0;
        const int jn = ring_slot(s, i + 1, m1);
        const V16 sn = ld16(Sb + jn * stride2, sgn);
        const V16 yn = ld16(Yb + jn * stride2, sgn);
        double a[6] = {dot16(sj, vs), dot16(sj, vy), dot16(sj, vg), dot16(yj, vs), dot16(yj, vy), dot16(yj, vg)};
        wave_sums(j, a);
        sj = sn;
        yj = yn;
    }
    __syncthreads();
    if (threadIdx.x < 6 * m1) {
        const int j = threadIdx.x / 6, back = h - 1 - j < 0 ? h - 1 - j + m1 : h - 1 - j;   // how many pairs ago
        const double *w = red[threadIdx.x];
        pp[threadIdx.x] = j == h || back < count ? ((w[0] + w[1]) + w[2]) + w[3] : 0.0;   // else: no pair
    }
}

// p = sum_b c_b v_b over the active basis {g, s_j, y_j : valid j} with the coefficients that the
// finalisation of the Gram pass left in coef[] (index 2 m1 for g, j for s_j, m1 + j for y_j).
__global__ __launch_bounds__(256) void combine_kernel(const VecSeg *__restrict__ segs, int m1,
                                                      float *__restrict__ p, const float *__restrict__ g,
                                                      const float *__restrict__ Sb, const float *__restrict__ Yb,
                                                      int64_t stride2, const SolveScalars *__restrict__ sc,
                                                      const double *__restrict__ coef, int64_t cstride) {
    const VecSeg sg = segs[blockIdx.x];
    const SolveScalars &s = sc[sg.prob];
    const double *c = coef + (int64_t)sg.prob * cstride;
    const int count = s.count;
    // FP32 vectors and FP32 accumulation (the coefficients come from the FP64 two-loop on the Gram
    // matrix and are rounded once to FP32), fixed order: g, then the pairs newest first
    V16 r;
    {
        const V16 vg = ld16(g, sg);
        const float cg = (float)c[2 * m1];
#pragma unroll
        for (int u = 0; u < 4 * VQ; ++u) r.v[u] = cg * vg.v[u];
    }
    for (int i = 0; i < count; ++i) {
        const int j = ring_slot(s, i, m1);
        const float cs = (float)c[j], cy = (float)c[m1 + j];
        const V16 sj = ld16(Sb + j * stride2, sg);
        const V16 yj = ld16(Yb + j * stride2, sg);
#pragma unroll
        for (int u = 0; u < 4 * VQ; ++u) r.v[u] = fmaf(cy, yj.v[u], fmaf(cs, sj.v[u], r.v[u]));
    }
    st16(p, sg, r);
}

// p = -g (steepest descent: first iteration, restarts of plain gradient descent)
__global__ __launch_bounds__(256) void negate_kernel(const VecSeg *__restrict__ segs, float *__restrict__ p,
                                                     const float *__restrict__ g) {
    const VecSeg sg = segs[blockIdx.x];
    V16 v = ld16(g, sg);
#pragma unroll
    for (int u = 0; u < 4 * VQ; ++u) v.v[u] = -v.v[u];
    st16(p, sg, v);
}

// g += 2 lambda (theta - c)   (c = 0 when cen is NULL)
__global__ __launch_bounds__(256) void reg_grad_kernel(const VecSeg *__restrict__ segs, float *__restrict__ g,
                                                       const float *__restrict__ th, const float *__restrict__ cen,
                                                       float lam2) {
    const VecSeg sg = segs[blockIdx.x];
    V16 v = ld16(g, sg);
    V16 t = ld16(th, sg);
    if (cen) {
        const V16 c = ld16(cen, sg);
#pragma unroll
        for (int u = 0; u < 4 * VQ; ++u) t.v[u] -= c.v[u];
    }
#pragma unroll
    for (int u = 0; u < 4 * VQ; ++u) v.v[u] += lam2 * t.v[u];
    st16(g, sg, v);
}

// penalty sums with d = theta - c (c = 0 when cen is NULL):
//   p == NULL: partial ||d||^2 ;   else partials Re<d, p>, ||p||^2
__global__ __launch_bounds__(256) void pen_kernel(const VecSeg *__restrict__ segs, const float *__restrict__ th,
                                                  const float *__restrict__ cen, const float *__restrict__ p,
                                                  double *__restrict__ part) {
    __shared__ double red[4 * 2];
    const VecSeg sg = segs[blockIdx.x];
    V16 d = ld16(th, sg);
    if (cen) {
        const V16 c = ld16(cen, sg);
#pragma unroll
        for (int u = 0; u < 4 * VQ; ++u) d.v[u] -= c.v[u];
    }
    if (!p) {
        double a[1] = {dot16(d, d)};
        block_sums<1>(a, red);
        if (threadIdx.x == 0) part[sg.part] = a[0];
        return;
    }
    const V16 vp = ld16(p, sg);
    double a[2] = {dot16(d, vp), dot16(vp, vp)};
    block_sums<2>(a, red);
    if (threadIdx.x == 0) { part[2 * sg.part] = a[0]; part[2 * sg.part + 1] = a[1]; }
}

// ADMM split and scaled dual (init: z = theta, u = 0), then the next X-update's center c = z - u:
//   z = (theta + u) * scale with scale = 1 / (1 + 2 lambda / rho);  u = u + theta - z
__global__ __launch_bounds__(256) void admm_update_kernel(const VecSeg *__restrict__ segs, int init,
                                                          const float *__restrict__ th, float *__restrict__ z,
                                                          float *__restrict__ uu, float *__restrict__ cen,
                                                          float scale) {
    const VecSeg sg = segs[blockIdx.x];
    const V16 t = ld16(th, sg);
    V16 vz, vu;
    if (init) {
        vz = t;
#pragma unroll
        for (int q = 0; q < 4 * VQ; ++q) vu.v[q] = 0.f;
    } else {
        vu = ld16(uu, sg);
#pragma unroll
        for (int q = 0; q < 4 * VQ; ++q) {
            vz.v[q] = (t.v[q] + vu.v[q]) * scale;
            vu.v[q] = vu.v[q] + t.v[q] - vz.v[q];
        }
    }
    st16(z, sg, vz);
    st16(uu, sg, vu);
#pragma unroll
    for (int q = 0; q < 4 * VQ; ++q) vz.v[q] -= vu.v[q];
    st16(cen, sg, vz);
}

// theta += step p, S[head] = step p (Sb not null); part (or null): ||theta - cen||^2 of the segment (cen null: 0)
__device__ __forceinline__ void theta_update(const VecSeg &sg, float *__restrict__ th, const float *__restrict__ p,
                                             float *__restrict__ Sb, int64_t stride2, const float *__restrict__ cen,
                                             const SolveScalars *__restrict__ sc, double *__restrict__ part, double *red) {
    // the vector loads need the segment only: they are in flight while the step is read
    V16 v = ld16(th, sg);
    V16 sp = ld16(p, sg);
    const SolveScalars &s = sc[sg.prob];
    const float a = (float)s.step;
    const bool frozen = s.frozen != 0;   // a non-finite step froze this problem: theta stays as is
#pragma unroll
    for (int u = 0; u < 4 * VQ; ++u) {
        sp.v[u] = a * sp.v[u];
        const float nv = v.v[u] + sp.v[u];
        v.v[u] = frozen ? v.v[u] : nv;
    }
    if (!frozen) {
        st16(th, sg, v);
        if (Sb) st16(Sb + s.head * stride2, sg, sp);
    }
    if (!part) return;
    if (cen) {
        const V16 c = ld16(cen, sg);
#pragma unroll
        for (int u = 0; u < 4 * VQ; ++u) v.v[u] -= c.v[u];
    }
    double acc[1] = {dot16(v, v)};
    block_sums<1>(acc, red);
    if (threadIdx.x == 0) part[sg.part] = acc[0];
}

// r += step a + step^2 b; part: |r|^2 of the segment
__device__ __forceinline__ void resid_update(const VecSeg &sg, float *__restrict__ r, const float *__restrict__ a,
                                             const float *__restrict__ b, const SolveScalars *__restrict__ sc,
                                             double *__restrict__ part, double *red) {
    // the vector loads need the segment only: they are in flight while the step is read
    V16 v = ld16(r, sg);
    const V16 va = ld16(a, sg), vb = ld16(b, sg);
    const SolveScalars &s = sc[sg.prob];
    // a non-finite step froze this problem: r stays as is (the update is discarded, nothing written)
    const bool frozen = s.frozen != 0;
    const float al = (float)s.step;
    const float al2 = (float)(s.step * s.step);
#pragma unroll
    for (int u = 0; u < 4 * VQ; ++u) {
        const float nv = v.v[u] + (al * va.v[u] + al2 * vb.v[u]);
        v.v[u] = frozen ? v.v[u] : nv;
    }
    if (!frozen) st16(r, sg, v);
    double acc[1] = {dot16(v, v)};
    block_sums<1>(acc, red);
    if (threadIdx.x == 0) part[sg.part] = acc[0];
}

__global__ __launch_bounds__(256) void theta_update_kernel(const VecSeg *__restrict__ segs, float *__restrict__ th,
                                                           const float *__restrict__ p, float *__restrict__ Sb,
                                                           int64_t stride2, const float *__restrict__ cen,
                                                           const SolveScalars *__restrict__ sc,
                                                           double *__restrict__ part) {
    __shared__ double red[4];
    theta_update(segs[blockIdx.x], th, p, Sb, stride2, cen, sc, part, red);
}

__global__ __launch_bounds__(256) void resid_update_kernel(const VecSeg *__restrict__ segs, float *__restrict__ r,
                                                           const float *__restrict__ a, const float *__restrict__ b,
                                                           const SolveScalars *__restrict__ sc,
                                                           double *__restrict__ part) {
    __shared__ double red[4];
    resid_update(segs[blockIdx.x], r, a, b, sc, part, red);
}

// both in one launch (no penalty term: the sums of theta are not wanted), the first nr blocks for r
__global__ __launch_bounds__(256) void update_kernel(const VecSeg *__restrict__ rsegs, int nr, const VecSeg *__restrict__ tsegs,
                                                     float *__restrict__ r, const float *__restrict__ a,
                                                     const float *__restrict__ b, float *__restrict__ th,
                                                     const float *__restrict__ p, float *__restrict__ Sb, int64_t stride2,
                                                     const SolveScalars *__restrict__ sc, double *__restrict__ part) {
    __shared__ double red[4];
    if ((int)blockIdx.x < nr) resid_update(rsegs[blockIdx.x], r, a, b, sc, part, red);
    else theta_update(tsegs[blockIdx.x - nr], th, p, Sb, stride2, nullptr, sc, nullptr, red);
}

// ---------------------------------------------------------------------------
// per-problem finalisation (one block per problem)
// ---------------------------------------------------------------------------
// the objective of one problem into its scalars and the history; rr = ||r||^2
__device__ __forceinline__ void record_f(const FinArgs &fa, int prob, double rr, SolveScalars &s) {
    const double f = 0.5 * rr + fa.lam * s.thnorm2;
    s.f = f;
    s.fdata = 0.5 * rr;
    if (fa.fhist) fa.fhist[prob][fa.t] = f;
    else if (fa.fhist0) fa.fhist0[fa.t] = f;
}

// One problem's partial sums, n to a slot, through a buffer as long as they are: what lies past the end reads zero, so
// the loads of several slots carry no conditions and are all in flight together.
constexpr uint32_t NO_SUM = 0xffffff00u;   // an offset past every end
__device__ __forceinline__ __amdgpu_buffer_rsrc_t sums_rsrc(const double *base, int count, int n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(base), (short)0, count * n * 8, 0x00020000);
}
__device__ __forceinline__ double ld_sum(__amdgpu_buffer_rsrc_t rs, uint32_t at) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, 0, 0));
}

// the sum of count partials by the first 256 threads, in thread 0 (the order of the products' sums in finalize_kernel)
__device__ __forceinline__ double first_sum(const double *base, int count, double *red) {
    const int t = threadIdx.x;
    if (t < 256) {
        const auto rs = sums_rsrc(base, count, 1);
        double v = 0.0;
        for (int i0 = t; i0 < count; i0 += 1024) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = ld_sum(rs, 8u * (uint32_t)(i0 + 256 * u));
#pragma unroll
            for (int u = 0; u < 4; ++u) v += x[u];
        }
        v = wave_sum64(v);
        if ((t & 63) == 0) red[t >> 6] = v;
    }
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ double of_lane(double v, int l) {   // l uniform
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | lo);
}

// Gram entries of the newest pair and of g, and the direction's coefficients: by one wave, lane i works for the i-th
// newest pair held. G: the staged Gram matrix nb x nb, then nb coefficients, basis (s_j, y_j, g).
__device__ __forceinline__ void gram_scalars(const FinArgs &fa, const double *tot, double *G, SolveScalars &s) {
    const int lane = threadIdx.x;
    const int m1 = fa.m1, nb = 2 * m1 + 1, ig = 2 * m1;
    double *cf = G + nb * nb;
    const int h = s.head;
    int head = h, cnt = s.count;
    double gamma = s.gamma;
    auto slot = [&](int i) {   // i < m1
        const int j = head - 1 - i;
        return j < 0 ? j + m1 : j;
    };
    const double *th = tot + 6 * h;
    const double sy = th[1], yy = th[2];
    const bool take = sy > 0.0 && yy > 0.0 && isfinite(sy) && isfinite(yy) && !s.frozen;
    if (lane < cnt) {
        const int j = slot(lane);
        const double *tj = tot + 6 * j;
        // g against the pairs already held (before the newest one is taken in)
        G[ig * nb + j] = G[j * nb + ig] = tj[2];
        G[ig * nb + m1 + j] = G[(m1 + j) * nb + ig] = tj[5];
        if (take) {
            G[j * nb + h] = G[h * nb + j] = tj[0];
            G[j * nb + m1 + h] = G[(m1 + h) * nb + j] = tj[1];
            G[(m1 + j) * nb + h] = G[h * nb + m1 + j] = tj[3];
            G[(m1 + j) * nb + m1 + h] = G[(m1 + h) * nb + m1 + j] = tj[4];
        }
    }
    if (take) {
        gamma = sy / yy;
        head = h + 1 == m1 ? 0 : h + 1;
        cnt = min(cnt + 1, m1 - 1);
    }
    if (lane == 0) {
        G[ig * nb + ig] = th[5];
        s.sy = sy;
        s.yy = yy;
        if (take) {
            G[h * nb + h] = th[0];
            G[h * nb + m1 + h] = G[(m1 + h) * nb + h] = sy;
            G[(m1 + h) * nb + m1 + h] = yy;
            G[ig * nb + h] = G[h * nb + ig] = th[3];
            G[ig * nb + m1 + h] = G[(m1 + h) * nb + ig] = th[4];
            s.rho[h] = 1.0 / sy;
        }
    }
    for (int b = lane; b < nb; b += 64) cf[b] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // the other lanes' entries
    // Two-loop recursion on coefficient vectors over the basis: q = sum_b d_b v_b, so <v_a, q> = sum_b G_ab d_b, the
    // pairs' terms formed by their lanes and added newest first. A row is read while the one before is worked on.
    struct Row {
        double s, y, g;
    };
    const bool mine = lane < cnt;
    const int j = mine ? slot(lane) : 0;
    const double rho = mine ? s.rho[j] : 0.0;
    double cs = 0.0, cy = 0.0, cg = 1.0, al = 0.0;
    auto row = [&](int a) {
        const double *r = G + a * nb;
        return Row{r[j], r[m1 + j], r[ig]};
    };
    auto dot = [&](const Row &r) {
        const double t = mine ? r.s * cs + r.y * cy : 0.0;
        double v = r.g * cg;
        for (int i = 0; i < cnt; ++i) v += of_lane(t, i);
        return v;
    };
    Row next = row(cnt > 0 ? slot(0) : ig);
    for (int i = 0; i < cnt; ++i) {   // newest first
        const Row r = next;
        next = row(i + 1 < cnt ? slot(i + 1) : m1 + slot(i));
        const double a = of_lane(rho, i) * dot(r);
        if (lane == i) {
            al = a;
            cy -= a;
        }
    }
    if (cnt > 0) {
        cy *= gamma;
        cg *= gamma;
    }
    for (int i = cnt - 1; i >= 0; --i) {   // oldest first
        const Row r = next;
        next = row(i > 0 ? m1 + slot(i - 1) : ig);
        const double beta = of_lane(rho, i) * dot(r);
        if (lane == i) cs += al - beta;
    }
    cs = -cs;
    cy = -cy;
    cg = -cg;
    double gp = dot(next);
    const bool restart = gp >= 0.0 || !isfinite(gp);
    if (restart) {   // not a descent direction: p = -g and the history is dropped
        cs = cy = 0.0;
        cg = -1.0;
        gp = -next.g;
    }
    if (mine) {
        cf[j] = cs;
        cf[m1 + j] = cy;
    }
    if (lane == 0) {
        cf[ig] = cg;
        s.head = head;
        s.count = restart ? 0 : cnt;
        s.gamma = restart ? 1.0 : gamma;
        s.restart = restart ? 1 : 0;
        s.gp = gp;
    }
}

// the scalar work of one problem (thread 0), all but the Gram pass's
__device__ __forceinline__ void finalize_scalars(const FinArgs &fa, int prob, const double *tot, SolveScalars &s) {
    switch (fa.op) {
        case FIN_F:
            record_f(fa, prob, tot[0], s);
            break;
        case FIN_F_OUT: {  // plain objective into fout[prob]
            if (fa.fout) fa.fout[prob] = 0.5 * tot[0];
            break;
        }
        case FIN_THNORM:
            s.thnorm2 = tot[0];
            break;
        case FIN_RECORD:  // data misfit of the tracked residual into the history at index t
            if (fa.fhist) fa.fhist[prob][fa.t] = s.fdata;
            else if (fa.fhist0) fa.fhist0[fa.t] = s.fdata;
            break;
        case FIN_RESET:  // fresh pair memory (a new sub-problem starts from the current theta)
            s.head = 0; s.count = 0; s.restart = 0; s.gamma = 1.0;
            break;
        case FIN_LAMTERMS:  // (Re<theta - c, p>, ||p||^2)
            s.tp = tot[0];
            s.pnorm2 = tot[1];
            break;
        case FIN_LINE: {  // tot = (Re<r,a>, |a|^2, Re<r,b>, Re<a,b>, |b|^2)
            double c[4];
            c[0] = tot[0] + 2.0 * fa.lam * s.tp;
            c[1] = tot[1] + 2.0 * tot[2] + 2.0 * fa.lam * s.pnorm2;
            c[2] = 3.0 * tot[3];
            c[3] = 2.0 * tot[4];
            for (int k = 0; k < 4; ++k) s.coef[k] = c[k];
            double a = exact_step_dev(c);
            bool bad = !isfinite(a);
            for (int k = 0; k < 4; ++k) bad = bad || !isfinite(c[k]);
            if (bad) s.frozen = 1;
            if (s.frozen) a = 0.0;
            s.step = a;
            break;
        }
        default: break;
    }
}

constexpr int FIN_NB = 2 * (MAX_LBFGS_M + 1) + 1;
constexpr int FIN_FEW = 5;
// One workgroup per problem: the sums, then the scalars by one thread, or the Gram pass's by one wave. The launch lies
// between two others that wait for it, so its latency is what counts: the loads of several slots are in flight
// together, the scalars are worked on in LDS (they are read and written there and in global memory by all threads at
// once), and the Gram pass's 6 m1 sums are added by 1024 threads (NT), each every (1024 / 6 m1)-th segment of one sum.
// us at nr 1024, tiles 128, of 4.7 that any launch in the chain takes: the line sums (1024 slots) 9.7 with a slot's
// loads after another's, now 4.6; Gram with none to four pairs held 10.5 to 14 by 256 threads in global memory, 6.6 to
// 8 with one thread's recursion, now 5.1 to 7.2.
template <int NT>
__global__ __launch_bounds__(NT) void finalize_kernel(FinArgs fa) {
    __shared__ double tot[6 * (MAX_LBFGS_M + 1)];
    __shared__ double sG[NT > 256 ? FIN_NB * FIN_NB + FIN_NB : 1];
    __shared__ double red[NT > 256 ? NT : 4 * FIN_FEW];
    __shared__ SolveScalars ss;
    static_assert(sizeof(SolveScalars) % 8 == 0 && sizeof(SolveScalars) / 8 <= 256, "one word per thread");
    constexpr int SW = sizeof(SolveScalars) / 8;
    const int prob = blockIdx.x;
    const int t = threadIdx.x;
    if constexpr (NT > 256) {
        if (blockIdx.y == 1) {   // the objective of the update before, beside the Gram sums: its two scalars only
            const double s = first_sum(fa.fpartials + (int64_t)prob * fa.pstride, fa.fcount, red);
            if (t == 0) record_f(fa, prob, s, fa.sc[prob]);
            return;
        }
    }
    const bool scalars = fa.op != FIN_F_OUT;   // the plain objective has none
    double *gs = reinterpret_cast<double *>(fa.sc + prob), *ls = reinterpret_cast<double *>(&ss);
    if (scalars && t < SW) ls[t] = gs[t];
    const int count = fa.counts ? fa.counts[prob] : fa.ucount;
    const auto rs = sums_rsrc(fa.partials + (int64_t)prob * fa.pstride * fa.nsum, count, fa.nsum);
    const int lane = t & 63, wv = t >> 6;
    if constexpr (NT == 256) {
        // products' sums, up to thousands of slots: a thread adds every 256th slot, all sums of a slot at once
        // (their loads are in flight together), then the lanes and the four waves
        double v[FIN_FEW];
#pragma unroll
        for (int k = 0; k < FIN_FEW; ++k) v[k] = 0.0;
        for (int i0 = t; i0 < count; i0 += 1024) {
            double x[4][FIN_FEW];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < FIN_FEW; ++k)
                    x[u][k] = ld_sum(rs, k < fa.nsum ? 8u * (uint32_t)((i0 + 256 * u) * fa.nsum + k) : NO_SUM);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < FIN_FEW; ++k) v[k] += x[u][k];
        }
#pragma unroll
        for (int k = 0; k < FIN_FEW; ++k) {
            if (k >= fa.nsum) break;
            const double s = wave_sum64(v[k]);
            if (lane == 0) red[wv * FIN_FEW + k] = s;
        }
        __syncthreads();
        if (t < fa.nsum)
            tot[t] = (red[t] + red[FIN_FEW + t]) + (red[2 * FIN_FEW + t] + red[3 * FIN_FEW + t]);
    } else {
        const int parts = NT / fa.nsum;   // fa.nsum <= 6 (MAX_LBFGS_M + 1)
        const int q = t / fa.nsum;
        double v = 0.0;
        for (int i0 = q; i0 < count; i0 += 8 * parts) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * parts;
                x[u] = ld_sum(rs, q < parts ? 8u * (uint32_t)(i * fa.nsum + (t - q * fa.nsum)) : NO_SUM);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) v += x[u];
        }
        red[t] = v;
        __syncthreads();
        if (t < fa.nsum) {
            double a = 0.0;
            for (int i0 = 0; i0 < parts; i0 += 8) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = red[i0 + u < parts ? (i0 + u) * fa.nsum + t : 0];
#pragma unroll
                for (int u = 0; u < 8; ++u) a += i0 + u < parts ? x[u] : 0.0;
            }
            tot[t] = a;
        }
    }
    const int m1 = fa.m1;
    const int gwords = (2 * m1 + 1) * (2 * m1 + 1) + 2 * m1 + 1;
    double *Gg = fa.gram + (int64_t)prob * fa.gstride;
    if constexpr (NT > 256)   // FIN_GRAM
        for (int i = t; i < gwords; i += NT) sG[i] = Gg[i];
    __syncthreads();
    if constexpr (NT > 256) {
        if (t < 64) gram_scalars(fa, tot, sG, ss);
    } else {
        if (t == 0) finalize_scalars(fa, prob, tot, ss);
    }
    __syncthreads();
    // (all but the objective, the first two, which the other workgroup may write)
    static_assert(offsetof(SolveScalars, f) == 0 && offsetof(SolveScalars, fdata) == 8, "the objective's words");
    if (scalars && t < SW && (NT == 256 || t > 1)) gs[t] = ls[t];
    if constexpr (NT > 256)
        for (int i = t; i < gwords; i += NT) Gg[i] = sG[i];
}


}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_stage_d(const float2 *D, int64_t ns, int64_t nr, float2 *Ds, int64_t ldk, int64_t lds, hipStream_t s) {
    dim3 grid((unsigned)((ldk + 31) / 32), (unsigned)((lds + 31) / 32));
    hipLaunchKernelGGL(stage_d_kernel, grid, dim3(256), 0, s, D, ns, nr, Ds, ldk, lds);
    return hipGetLastError();
}

hipError_t launch_stage_d_split(const Problems &in, int count, int64_t ns, int64_t nr, uint32_t *Dh, uint32_t *Dl,
                                int64_t ldk, uint32_t *DHh, uint32_t *DHl, int64_t lds, int64_t stride, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (ldk % 32 || lds % 32 || count > PROBLEMS_MAX) return hipErrorInvalidValue;   // whole blocks
    dim3 grid((unsigned)(ldk / 32), (unsigned)(lds / 32), (unsigned)count);
    hipLaunchKernelGGL(stage_d_split_kernel, grid, dim3(256), 0, s, in, ns, nr, Dh, Dl, ldk, DHh, DHl, lds, stride);
    return hipGetLastError();
}

namespace {
unsigned theta_blocks(const Problems &in, int count) {
    int64_t n = 1;
    for (int p = 0; p < count; ++p) n = std::max(n, in.theta_n[p]);
    return (unsigned)((n + 1023) / 1024);
}
}  // namespace

hipError_t launch_stage_problems(const Problems &in, int count, int64_t ns, int64_t nr, int64_t lds, int64_t ldk,
                                 float2 *Ds, float2 *Us, const ProbOff *probs, float2 *th, SolveScalars *sc,
                                 hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (lds % STG_ROWS || count > PROBLEMS_MAX) return hipErrorInvalidValue;
    const unsigned rows = (unsigned)(lds / STG_ROWS) * ((Ds ? 1u : 0u) + (Us ? 1u : 0u));
    hipLaunchKernelGGL(stage_problems_kernel, dim3(rows + theta_blocks(in, count), (unsigned)count), dim3(256), 0, s, in,
                       ns, nr, lds, ldk, Ds, Us, probs, th, sc);
    return hipGetLastError();
}

hipError_t launch_collect_theta(const Problems &out, int count, const ProbOff *probs, const float2 *th, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (count > PROBLEMS_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(collect_theta_kernel, dim3(theta_blocks(out, count), (unsigned)count), dim3(256), 0, s, out, probs,
                       th);
    return hipGetLastError();
}

hipError_t launch_split_transpose(const float2 *r, int64_t ldr, int64_t rows, int64_t cols, uint32_t *th,
                                  uint32_t *tl, int64_t rowsp, int64_t colsp, int batch, int64_t s_r, int64_t s_t,
                                  hipStream_t s) {
    if (rows <= 0 || cols <= 0 || batch <= 0) return hipSuccess;
    if (rowsp % 32 || colsp % 32 || rowsp < rows || colsp < cols) return hipErrorInvalidValue;   // whole blocks
    dim3 grid((unsigned)(colsp / 32), (unsigned)(rowsp / 32), (unsigned)batch);
    hipLaunchKernelGGL(split_transpose_kernel, grid, dim3(256), 0, s, r, ldr, rows, cols, th, tl, rowsp, s_r, s_t);
    return hipGetLastError();
}

hipError_t launch_zero_pad(uint32_t *base, int64_t ld, int64_t n, int nplanes, int64_t plane_stride, int batch,
                           int64_t batch_stride, hipStream_t s) {
    if (ld <= n || nplanes <= 0 || batch <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_pad_kernel, dim3((unsigned)ld, (unsigned)nplanes, (unsigned)batch), dim3(128), 0, s, base, ld,
                       n, plane_stride, batch_stride);
    return hipGetLastError();
}

hipError_t launch_copy2d(const float2 *src, int64_t lds, float2 *dst, int64_t ldd, int64_t rows,
                         int64_t cols, hipStream_t s) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const unsigned gx = (unsigned)std::min<int64_t>((cols + 255) / 256, 64);
    const unsigned gy = (unsigned)std::min<int64_t>(rows, 65535);
    hipLaunchKernelGGL(copy2d_kernel, dim3(gx, gy), dim3(256), 0, s, src, lds, dst, ldd, rows, cols);
    return hipGetLastError();
}

hipError_t launch_permute_cols(const float2 *in, const int64_t *perm, float2 *out, int64_t rows,
                               int64_t cols, int32_t *bad, hipStream_t s) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const unsigned gx = (unsigned)std::min<int64_t>((cols + 255) / 256, 64);
    const unsigned gy = (unsigned)std::min<int64_t>(rows, 65535);
    hipLaunchKernelGGL(permute_kernel, dim3(gx, gy), dim3(256), 0, s, in, perm, out, rows, cols, bad);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (((uintptr_t)p & 3) || (bytes & 3)) return hipErrorInvalidValue;
    const int64_t words = (int64_t)(bytes / 4);
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>((words / 4 + 255) / 256, 4096));
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, (uint32_t *)p, words);
    return hipGetLastError();
}

#define SEGS_LAUNCH(kern, nseg, s, ...)                                              \
    do {                                                                             \
        if ((nseg) <= 0) return hipSuccess;                                          \
        hipLaunchKernelGGL(kern, dim3((unsigned)(nseg)), dim3(256), 0, s, __VA_ARGS__); \
        return hipGetLastError();                                                    \
    } while (0)

hipError_t launch_gram(const VecSeg *segs, int nseg, int m1, const float *g, const float *gprev, float *Yb,
                       const float *Sb, int64_t stride2, const SolveScalars *sc, double *part, hipStream_t s) {
    SEGS_LAUNCH(gram_kernel, nseg, s, segs, m1, g, gprev, Yb, Sb, stride2, sc, part);
}
hipError_t launch_combine(const VecSeg *segs, int nseg, int m1, float *p, const float *g, const float *Sb,
                          const float *Yb, int64_t stride2, const SolveScalars *sc, const double *coef,
                          int64_t cstride, hipStream_t s) {
    SEGS_LAUNCH(combine_kernel, nseg, s, segs, m1, p, g, Sb, Yb, stride2, sc, coef, cstride);
}
hipError_t launch_negate(const VecSeg *segs, int nseg, float *p, const float *g, hipStream_t s) {
    SEGS_LAUNCH(negate_kernel, nseg, s, segs, p, g);
}
hipError_t launch_reg_grad(const VecSeg *segs, int nseg, float *g, const float *th, const float *cen, float lam2,
                           hipStream_t s) {
    SEGS_LAUNCH(reg_grad_kernel, nseg, s, segs, g, th, cen, lam2);
}
hipError_t launch_pen(const VecSeg *segs, int nseg, const float *th, const float *cen, const float *p, double *part,
                      hipStream_t s) {
    SEGS_LAUNCH(pen_kernel, nseg, s, segs, th, cen, p, part);
}
hipError_t launch_admm_update(const VecSeg *segs, int nseg, int init, const float *th, float *z, float *u, float *cen,
                              float scale, hipStream_t s) {
    SEGS_LAUNCH(admm_update_kernel, nseg, s, segs, init, th, z, u, cen, scale);
}
hipError_t launch_theta_update(const VecSeg *segs, int nseg, float *th, const float *p, float *Sb,
                               int64_t stride2, const float *cen, const SolveScalars *sc, double *part,
                               hipStream_t s) {
    SEGS_LAUNCH(theta_update_kernel, nseg, s, segs, th, p, Sb, stride2, cen, sc, part);
}
hipError_t launch_resid_update(const VecSeg *segs, int nseg, float *r, const float *a, const float *b,
                               const SolveScalars *sc, double *part, hipStream_t s) {
    SEGS_LAUNCH(resid_update_kernel, nseg, s, segs, r, a, b, sc, part);
}
hipError_t launch_update(const VecSeg *rsegs, int nrseg, const VecSeg *tsegs, int ntseg, float *r, const float *a,
                         const float *b, float *th, const float *p, float *Sb, int64_t stride2, const SolveScalars *sc,
                         double *part, hipStream_t s) {
    if (nrseg + ntseg <= 0) return hipSuccess;
    hipLaunchKernelGGL(update_kernel, dim3((unsigned)(nrseg + ntseg)), dim3(256), 0, s, rsegs, nrseg, tsegs, r, a, b, th, p,
                       Sb, stride2, sc, part);
    return hipGetLastError();
}
hipError_t launch_finalize(const FinArgs &fa, int nprob, hipStream_t s) {
    if (nprob <= 0) return hipSuccess;
    if ((fa.op == FIN_GRAM) != (fa.nsum > FIN_FEW) || fa.nsum > 6 * (MAX_LBFGS_M + 1)) return hipErrorInvalidValue;
    if (fa.op == FIN_GRAM) hipLaunchKernelGGL(finalize_kernel<1024>, dim3((unsigned)nprob, fa.fpartials ? 2 : 1), dim3(1024), 0, s, fa);
    else hipLaunchKernelGGL(finalize_kernel<256>, dim3((unsigned)nprob), dim3(256), 0, s, fa);
    return hipGetLastError();
}

}  // namespace tlr
