// Device arithmetic shared by the Lanczos kernels: every kernel evaluates
// these expressions identically, so a column's vectors do not depend on
// which of them ran.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vne {

// Lazily normalised Lanczos vector: v_j = (P_j - alpha_{j-1} v_{j-1}) / beta_{j-1},
// evaluated identically wherever an entry of v_j is needed.
__device__ __forceinline__ float materialize(float p, float vp, float a, float inv) {
    return __fmul_rn(__fmaf_rn(-a, vp, p), inv);
}
__device__ __forceinline__ double materialize(double p, double vp, double a, double inv) {
    return __dmul_rn(__fma_rn(-a, vp, p), inv);
}

// SplitMix64 output function (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t splitmix64_mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Rademacher entry for (row key, hash column): sign of the top bit of
// mix(seed + (key * 2^32 + col + 1) * 0x9E3779B97F4A7C15).
__device__ __forceinline__ double rademacher(uint64_t seed, int64_t key, int64_t col) {
    const uint64_t ctr = ((uint64_t)key << 32) + (uint64_t)col + 1ull;
    const uint64_t h = splitmix64_mix(seed + ctr * 0x9E3779B97F4A7C15ull);
    return (h >> 63) ? -1.0 : 1.0;
}

}  // namespace vne
