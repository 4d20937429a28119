// Cross-lane exchanges of 64-bit values inside a 64-lane wavefront (gfx950): DPP
// permutations of the Legendre adjoint and of the coefficient rotation.
#pragma once

#include <hip/hip_runtime.h>

namespace psht {

// x from lane i ^ 1 of the quad.
__device__ inline double quad_xor1(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0xB1, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0xB1, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Lane N of each 16-lane row of x, in every lane of the row (the one DPP
// permutation that moves 64-bit values, at full rate).
template <int N> __device__ inline double row_bcast(double x) {
    return __builtin_amdgcn_mov_dpp(x, 0x150 + N, 0xF, 0xF, false);
}

// Each 16-lane row of x rotated by 8 lanes: lane i gets lane i ^ 8.
__device__ inline double row_rotate8(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x128, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x128, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

}  // namespace psht
