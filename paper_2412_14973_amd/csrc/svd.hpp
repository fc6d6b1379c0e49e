// Batched per-tile FP64 SVD (one-sided Jacobi) for the rank estimate and the warm start (internal).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace tlr {

// One tile of X at (row0, col0), decomposed as A = X_ij (trans = 0) or A = X_ij^T (trans = 1, used
// when X_ij has fewer rows than columns, so that A is never wide); A is m x n. W and V are complex128
// column-major per tile.
struct SvdTile {
    int32_t m, n;    // rows / columns of A
    int32_t trans;
    int32_t grid;    // of several grids in one list of tiles (counts): which
    int64_t row0, col0;
    int64_t offW;    // W: m x n
    int64_t offV;    // V: n x n (warm start of a factored tile), -1 without V
    int64_t offS;    // sigma / order: n entries
    int32_t npad;    // n rounded up to even (round-robin players)
    int32_t pair0;   // first block of this tile in a round launch (prefix sum of npad / 2)
};

enum WarmKind : int32_t { WARM_LR = 0, WARM_QQ = 1, WARM_DENSE = 2 };
struct WarmItem {
    int32_t tile;    // SvdTile index
    int32_t kind;    // WarmKind
    int32_t k;       // rank kept
    int32_t pad;
    int64_t offA;    // theta offset of L / Q / Z
    int64_t offB;    // theta offset of R (LR)
};

constexpr int SVD_MAX_N = 1024;     // tile columns handled by the per-tile sort
constexpr int SVD_MAX_SWEEPS = 30;  // sweeps enqueued; converged sweeps return at once
constexpr double SVD_TOL = 1e-13;   // rotate a pair while |w_p^H w_q| > tol ||w_p|| ||w_q||

// nonfinite (may be NULL): set to 1 where a tile holds a value that is not finite
hipError_t launch_svd_gather(const SvdTile *tiles, int ntiles, const float2 *X, int64_t ldx, double2 *W, double2 *V,
                             int32_t *nonfinite, hipStream_t s);
hipError_t launch_svd_round(const SvdTile *tiles, const int32_t *pair_tile, int npairs, int round, double2 *W,
                            double2 *V, const int32_t *flags, int32_t *busy, double tol, hipStream_t s);
hipError_t launch_svd_sweep_end(int32_t *flags, int32_t *busy, hipStream_t s);
hipError_t launch_svd_sigma(const SvdTile *tiles, int ntiles, const double2 *W, double *sig, hipStream_t s);
hipError_t launch_svd_rank(const SvdTile *tiles, int ntiles, const double *sig, int64_t nsig, double eps,
                           int32_t *kout, double *v0out, hipStream_t s);
hipError_t launch_svd_order(const SvdTile *tiles, int ntiles, const double *sig, int32_t *order, hipStream_t s);
hipError_t launch_svd_factors(const SvdTile *tiles, const WarmItem *items, int nitems, const double2 *W,
                              const double2 *V, const double *sig, const int32_t *order, const float2 *X,
                              int64_t ldx, float2 *theta, hipStream_t s);

// Counts without vectors (bidiag.hip), tiles of at most BIDIAG_MAX_M rows (mmax: the largest). Up to 128 rows the
// tiles are read from X, else from W (gathered before). The squares of the bidiagonal go to d2 (sigma slots) and,
// with the tile's largest singular value, to the start of its W. mixed: tiles of several grids, all of which
// bidiag_shared() says can share a launch.
// BIDIAG_MAX_M: all ranks of a matrix against the rotations, ms: nr 1024 tiles of 257 9.4 and 35.6, 320 13.9 and 46.6, 448
// 25.9 and 74.0, 512 33.3 and 91.5; one tile of 300 12.3 and 27.2, one of 512 33.2 and 67.9; nr 4096 tiles of 512 36.1
// and 430. (Above 256 rows 63 of a lane's registers are spilled, up to there none.)
constexpr int BIDIAG_MAX_M = 512;
bool bidiag_reads_x(int mmax);
bool bidiag_shared(int64_t mmax);
hipError_t launch_bidiag(const SvdTile *tiles, int ntiles, bool mixed, int mmax, const float2 *X, int64_t ldx, double2 *W,
                         double *d2, int32_t *nonfinite, hipStream_t s);
// v0 = the largest of them, k = #{sigma >= eps v0} per tile, for each of ngrids lists of tiles: list g goes from
// first[g] to first[g + 1] (first null: one list)
hipError_t launch_svd_counts(const SvdTile *tiles, int ntiles, const int32_t *first, int ngrids, const double2 *W,
                             const double *d2, double eps, int32_t *kout, double *v0, hipStream_t s);

}  // namespace tlr
