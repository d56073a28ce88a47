// lanes.hpp -- lane exchanges in the VALU (moves within 16 lanes, swaps of 16
// or 32 lanes), float and double: a butterfly of __shfl_xor is a chain of
// LDS-crossbar round trips, six for every row a wave walks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rk {

template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int kQuadXor1 = 0xb1;     // lane ^ 1 (quad permutation 1 0 3 2)
constexpr int kQuadXor2 = 0x4e;     // lane ^ 2 (quad permutation 2 3 0 1)
constexpr int kHalfMirror = 0x141;  // 7 - lane within 8 lanes
constexpr int kRowMirror = 0x140;   // 15 - lane within 16 lanes
constexpr int kRor4 = 0x124, kRor8 = 0x128;     // rotations within 16 lanes

// v plus the value 16 (32) lanes away: swapping the odd 16-lane rows of one
// copy with the even rows of another (the upper half with the lower) leaves
// the two addends side by side.
__device__ __forceinline__ float add_row16(float v)
{
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ __forceinline__ double add_row16(double v)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ float add_half32(float v)
{
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ __forceinline__ double add_half32(double v)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

}  // namespace rk
