// wave.hpp -- wavefront helpers shared by the sweep kernels: a lane's column,
// whole-wavefront shifts and the open boundaries' data.
#pragma once

#include "kernels.hpp"

namespace trt {

namespace {

// Per-lane geometry of one strip column.
struct Column {
    int xm, xc, xp;        // wrapped columns x-1, x, x+1
    uint32_t om, oc, op;   // their byte offsets within a row
};

__device__ __forceinline__ Column column_of(int c, int nx, uint32_t elem) {
    Column col;
    col.xc = c % nx;
    if (col.xc < 0) col.xc += nx;
    col.xm = (col.xc == 0) ? nx - 1 : col.xc - 1;
    col.xp = (col.xc == nx - 1) ? 0 : col.xc + 1;
    col.om = (uint32_t)col.xm * elem;
    col.oc = (uint32_t)col.xc * elem;
    col.op = (uint32_t)col.xp * elem;
    return col;
}

// Boundary data of open x boundaries, in the arithmetic precision.
template <class C> struct OpenX {
    bool on;
    int nx;
    C u_in, rho_in, rho_out, phi_wall;
};

// DPP whole-wavefront shifts: lane i receives lane i-1 (shr) or lane i+1
// (shl); the lane with no source keeps `old`.
__device__ __forceinline__ float dpp_shr(float old, float src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                                  __builtin_bit_cast(int, src),
                                                                  0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float dpp_shl(float old, float src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                                  __builtin_bit_cast(int, src),
                                                                  0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ uint32_t dpp_shr(uint32_t old, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t dpp_shl(uint32_t old, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ double dpp_shr(double old, double src) {
    const uint64_t o = __builtin_bit_cast(uint64_t, old), v = __builtin_bit_cast(uint64_t, src);
    const uint32_t lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)v, 0x138, 0xf,
                                                    0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(v >> 32),
                                                    0x138, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double dpp_shl(double old, double src) {
    const uint64_t o = __builtin_bit_cast(uint64_t, old), v = __builtin_bit_cast(uint64_t, src);
    const uint32_t lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)v, 0x130, 0xf,
                                                    0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(v >> 32),
                                                    0x130, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The same shifts with zero in the lane that has no source: without a value to
// keep, the destination needs no move ahead of the shift (two per double), and
// the shift can become an operand modifier of its one use (a row of the
// three-step FP64 pipeline: 445 -> 409 vector instructions).  us per step, with
// the moves / without, in turn on one box: 4096^2 FP32 87.9 / 87.3, FP16 72.6 /
// 72.3, 2048^2 FP64 48.5 / 48.3, a 1050^2 FP64 cylinder 16.7 / 16.5; lanes without
// a source feed no stored column either way.
__device__ __forceinline__ uint32_t dpp_shr0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t dpp_shl0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);
}
__device__ __forceinline__ float dpp_shr0(float v) {
    return __builtin_bit_cast(float, dpp_shr0(__builtin_bit_cast(uint32_t, v)));
}
__device__ __forceinline__ float dpp_shl0(float v) {
    return __builtin_bit_cast(float, dpp_shl0(__builtin_bit_cast(uint32_t, v)));
}
__device__ __forceinline__ double dpp_shr0(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, ((uint64_t)dpp_shr0((uint32_t)(b >> 32)) << 32) |
                                          dpp_shr0((uint32_t)b));
}
__device__ __forceinline__ double dpp_shl0(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, ((uint64_t)dpp_shl0((uint32_t)(b >> 32)) << 32) |
                                          dpp_shl0((uint32_t)b));
}

// A wave-uniform value in scalar registers.
__device__ __forceinline__ float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

}  // namespace

}  // namespace trt
