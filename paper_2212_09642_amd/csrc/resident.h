// Launch of the on-chip Lanczos kernel (resident.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"
#include "resident_layout.h"

namespace vne {

constexpr size_t kResidentLds = 160 * 1024;   // LDS of a CU
// columns per workgroup times rounds: a lane keeps that many entries of
// v_{j-1} (or of w) in registers
constexpr int kResidentSlots32 = 39, kResidentSlots64 = 19;

// One matrix and its probe block; device pointers.
struct ResidentJob {
    const int4 *slices;
    const uint32_t *words;
    const void *vals;           // float2 / double2 per word (not unit)
    const int2 *spans;
    const int32_t *row_of;
    const double *diag;         // unit
    const int64_t *keys;
    const int32_t *colors;
    const void *dense;
    double *alpha, *beta;       // [columns][ld_k]
    double *norm2;
    int32_t *k_eff;
    int32_t *flags;
    uint64_t seed;
    double scale, off_value, tau;
    int32_t gen, ld_dense, desing, col_offset;
    int32_t n, m, k, ld_k, rounds, positions;
};

// LDS bytes of a workgroup
size_t resident_lds(int positions, int cols, bool fp64);

// Which kernel: columns per workgroup (1, 2 or 4; FP64: 1 or 2), equal
// off-diagonal values, element type, and whether a lane's slots need the
// large vectors.
struct ResidentKind {
    int cols;
    bool unit, fp64, big;
    bool operator==(const ResidentKind &o) const {
        return cols == o.cols && unit == o.unit && fp64 == o.fp64 && big == o.big;
    }
};
ResidentKind resident_kind(int rounds, int cols, bool unit, bool fp64);

// One matrix: a workgroup per group of kind.cols columns, m columns in all.
hipError_t launch_resident_one(const ResidentJob &job, int waves, const ResidentKind &kind, hipStream_t s);
// Several matrices of one number of waves and one kind: map entries {job,
// first column} ({-1, 0}: none); lds: the largest resident_lds of the jobs.
hipError_t launch_resident_many(const ResidentJob *jobs, const int2 *map, int32_t entries, int waves,
                                const ResidentKind &kind, size_t lds, hipStream_t s);

}  // namespace vne
