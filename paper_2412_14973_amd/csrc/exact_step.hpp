// Exact line-search step (internal): the positive minimiser of the quartic phi whose derivative is
// phi'(a) = c0 + c1 a + c2 a^2 + c3 a^3 (ADMM solver, X-update: f(theta + a p) is a quartic in a
// because C is quadratic in the factors). Host and device share this code; a CPU test program
// compares it with the oracle's root selection.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

namespace tlr {

using std::fabs;
using std::fmax;
using std::fmin;
using std::isfinite;
using std::sqrt;

__host__ __device__ inline double phi_inc(const double *c, double a) {
    return a * (c[0] + a * (c[1] / 2 + a * (c[2] / 3 + a * c[3] / 4)));
}

__host__ __device__ inline double dphi(const double *c, double a) { return ((c[3] * a + c[2]) * a + c[1]) * a + c[0]; }
__host__ __device__ inline double ddphi(const double *c, double a) { return (3.0 * c[3] * a + 2.0 * c[2]) * a + c[1]; }

// The root of phi' between x1 and x2, where phi' is monotone and phi'(x1), phi'(x2) have opposite
// signs: safeguarded Newton-Raphson (a Newton step is taken while it stays inside the bracket and
// at least halves the step before it; otherwise the bracket is bisected), converging to full
// precision without the cancellation of closed-form cubic roots.
__host__ __device__ inline double bracketed_root(const double *c, double x1, double x2) {
    const double f1 = dphi(c, x1), f2 = dphi(c, x2);
    if (f1 == 0.0) return x1;
    if (f2 == 0.0) return x2;
    double neg = f1 < 0.0 ? x1 : x2, pos = f1 < 0.0 ? x2 : x1;   // phi'(neg) < 0 < phi'(pos)
    double x = 0.5 * (x1 + x2), dx_old = fabs(x2 - x1), dx = dx_old;
    double f = dphi(c, x), fd = ddphi(c, x);
    for (int it = 0; it < 400; ++it) {
        const bool leaves = ((x - pos) * fd - f) * ((x - neg) * fd - f) > 0.0;
        const bool slow = fabs(2.0 * f) > fabs(dx_old * fd);
        dx_old = dx;
        if (leaves || slow) {
            dx = 0.5 * (pos - neg);
            x = neg + dx;
            if (x == neg) return x;
        } else {
            dx = f / fd;
            const double prev = x;
            x -= dx;
            if (x == prev) return x;
        }
        if (fabs(dx) <= 2.220446049250313e-16 * fabs(x)) return x;
        f = dphi(c, x);
        fd = ddphi(c, x);
        if (f == 0.0) return x;
        if (f < 0.0) neg = x;
        else pos = x;
    }
    return x;
}

// Positive minimiser of phi: the positive real root of phi' with the lowest phi (ties: the smaller
// step; none: 0). (0, inf) is split at the positive roots of phi'' into pieces on which phi' is
// monotone; each piece holds at most one root, found by bracketed_root (the last piece's bracket
// by doubling until phi' changes sign). A stationary point of phi' at which phi' vanishes (a double
// root) is a root too.
__host__ __device__ inline double exact_step_dev(const double *c) {
    const double scale = fabs(c[0]) + fabs(c[1]) + fabs(c[2]) + fabs(c[3]);
    if (!(scale > 0.0) || !isfinite(scale)) return 0.0;
    // positive roots of phi''(a) = c1 + 2 c2 a + 3 c3 a^2, ascending (stable quadratic formula)
    double brk0 = 0.0, brk1 = 0.0;
    int nb = 0;
    if (c[3] != 0.0) {
        const double disc = c[2] * c[2] - 3.0 * c[3] * c[1];
        if (disc > 0.0) {
            const double q = -(c[2] + (c[2] >= 0.0 ? sqrt(disc) : -sqrt(disc)));
            const double r1 = q / (3.0 * c[3]), r2 = q != 0.0 ? c[1] / q : r1;
            const double lo = fmin(r1, r2), hi = fmax(r1, r2);
            if (lo > 0.0 && isfinite(lo)) {
                brk0 = lo;
                nb = 1;
            }
            if (hi > 0.0 && isfinite(hi) && hi != lo) {
                (nb ? brk1 : brk0) = hi;
                ++nb;
            }
        }
    } else if (c[2] != 0.0) {
        const double r = -c[1] / (2.0 * c[2]);
        if (r > 0.0 && isfinite(r)) {
            brk0 = r;
            nb = 1;
        }
    }
    // sign of phi' as a -> inf: its leading nonzero coefficient
    const double lead = c[3] != 0.0 ? c[3] : c[2] != 0.0 ? c[2] : c[1] != 0.0 ? c[1] : c[0];
    double lo = 0.0, best = 0.0, bestv = 0.0;
    bool have = false;
    // One piece after the other through the same code: on the device a launch runs it once, so fetching it is much of
    // what it costs (the finalisation that holds it, nr 64: 6.5 to 7.2 us unrolled, 4.5 to 5.1 so).
#pragma unroll 1
    for (int k = 0; k <= nb; ++k) {
        const double hi = k == 0 ? brk0 : brk1;   // of all pieces but the last
        const double flo = dphi(c, lo);
        double x = 0.0;   // the piece's root
        if (k > 0 && flo == 0.0) {   // a root at a stationary point of phi'
            x = lo;
        } else {
            double x1 = lo, x2 = hi;
            bool bracket = false;
            if (k < nb) {
                const double fhi = dphi(c, hi);
                bracket = fhi != 0.0 && (flo < 0.0) != (fhi < 0.0) && flo != 0.0;
            } else if (flo != 0.0 && (flo < 0.0) != (lead < 0.0)) {   // last piece [lo, inf)
                x2 = lo > 0.0 ? 2.0 * lo : 1.0;
                double f2 = dphi(c, x2);
                int it = 0;
                while (isfinite(x2) && (f2 < 0.0) == (flo < 0.0) && f2 != 0.0 && it < 2200) {
                    x1 = x2;
                    x2 *= 2.0;
                    f2 = dphi(c, x2);
                    ++it;
                }
                bracket = isfinite(x2) && ((f2 < 0.0) != (flo < 0.0) || f2 == 0.0);
            }
            if (bracket) x = bracketed_root(c, x1, x2);
        }
        if (x > 0.0 && isfinite(x)) {
            const double v = phi_inc(c, x);
            if (!have || v < bestv || (v == bestv && x < best)) {
                best = x;
                bestv = v;
                have = true;
            }
        }
        lo = hi;
    }
    return have ? best : 0.0;
}

}  // namespace tlr
