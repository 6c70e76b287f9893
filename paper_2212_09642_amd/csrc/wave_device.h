// Wavefront and workgroup primitives of the on-chip kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vne {

// v + (v of the lane that the DPP control names; 0 where there is none)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// sum over the 64 lanes in lane 63: within rows of 16 lanes, then across
__device__ __forceinline__ double wave_total(double v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ double from_lane(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Barrier of the workgroup for LDS only: loads in flight (the next slice's
// words) and stores of the coefficients are not waited for, as the
// workgroup-wide fence of __syncthreads would; nothing in device memory
// passes between waves here.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// base + half-word H of w times SIZE, in one instruction
template <int H, int SIZE>
__device__ __forceinline__ uint32_t half_times(uint32_t w, uint32_t base) {
    uint32_t r;
    if (H == 0) asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(w), "n"(SIZE), "s"(base));
    else asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(w), "n"(SIZE), "s"(base));
    return r;
}

// device memory and LDS by their address spaces: a pointer that a kernel
// reads from memory is a generic one, whose loads take the LDS path too
#define VNE_GLOBAL __attribute__((address_space(1)))
#define VNE_LDS __attribute__((address_space(3)))
template <typename T>
__device__ __forceinline__ const VNE_GLOBAL T *global(const void *p) {
    return (const VNE_GLOBAL T *)(uintptr_t)p;
}

}  // namespace vne
