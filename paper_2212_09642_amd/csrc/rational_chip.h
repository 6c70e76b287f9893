// Rational Arnoldi steps of small matrices, one workgroup per column
// (rational_chip.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vne {

constexpr int kRChipRounds = 5;        // rounds of 1024 rows a workgroup takes

// The matrix in the on-chip layout (resident_layout.h) and the vectors of
// the run, per column and in position order: V [cols][kb][positions],
// U and W [cols][positions].
struct RChip {
    const int32_t *slices;
    const uint32_t *words;
    const double *vals;                // two per word (not unit)
    const int32_t *spans;
    const int32_t *row_of;
    const double *diag;                // unit
    double scale, off_value;
    int32_t waves, rounds, positions, word_rows;
    bool unit;
    int32_t kb, cols;
    double *V, *U, *W;
};

// v_1 = c / ||c|| (or 0) from the probe block W0 [n][mp]
hipError_t launch_rchip_start(const RChip &a, const double *W0, int32_t mp, const double *norm2, hipStream_t s);
// u = A v_j, and row and column j of every column's H [kb][kb]
hipError_t launch_rchip_project(const RChip &a, int32_t j, double *H, hipStream_t s);
// w = the solution of (I - A / xi) w = u by conjugate gradients, or u where xi = 0
hipError_t launch_rchip_solve(const RChip &a, const double *xi, double tol2, int32_t cg_max, int32_t *iters,
                              int64_t *apps, hipStream_t s);
// w (from_u: u) orthogonalized twice against v_1 .. v_j, ||w||^2 before and
// after; commit: v_{j+1} and the basis size too
hipError_t launch_rchip_orthogonalize(const RChip &a, int32_t j, bool from_u, bool commit, double *ww, double *ww0,
                                      int32_t *ke, hipStream_t s);
hipError_t launch_rchip_commit(const RChip &a, int32_t j, const double *ww, const double *ww0, int32_t *ke,
                               hipStream_t s);

}  // namespace vne
