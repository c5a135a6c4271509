// Sum over the 64 lanes of a wavefront, the same value in every lane, without LDS: data-parallel moves inside rows of 16 lanes
// (neighbours, pairs, mirrored halves, mirrored row), then the four rows' last lanes as scalars, in a fixed order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kavg {

template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float dpp_wave_sum(float x) {
    x += dpp_move<0xB1>(x);        // quad_perm [1,0,3,2]
    x += dpp_move<0x4E>(x);        // quad_perm [2,3,0,1]
    x += dpp_move<0x141>(x);       // row_half_mirror
    x += dpp_move<0x140>(x);       // row_mirror
    const int xi = __builtin_bit_cast(int, x);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 15));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 31));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 47));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 63));
    return (r0 + r1) + (r2 + r3);
}

// (r0 + r1) + (r2 + r3) over the four rows of 16 lanes, for each of the sixteen places of a row
__device__ __forceinline__ float rows_sum(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    x = __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return __builtin_bit_cast(float, (uint32_t)h[0]) + __builtin_bit_cast(float, (uint32_t)h[1]);
}

// op over the 64 lanes in the order of a butterfly over lane ^ 32, 16, 8, 4, 2, 1, every lane with the result: the halves and the
// rows are exchanged by swaps; from then on values repeat, so that rotations inside a row stand for lane ^ 8 and lane ^ 4.
template <class Op>
__device__ __forceinline__ float butterfly(float x, Op op) {
    auto bits = [](float v) { return __builtin_bit_cast(uint32_t, v); };
    const auto h = __builtin_amdgcn_permlane32_swap(bits(x), bits(x), false, false);
    x = op(__builtin_bit_cast(float, (uint32_t)h[0]), __builtin_bit_cast(float, (uint32_t)h[1]));
    const auto r = __builtin_amdgcn_permlane16_swap(bits(x), bits(x), false, false);
    x = op(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
    x = op(x, dpp_move<0x128>(x));             // row_ror:8
    x = op(x, dpp_move<0x124>(x));             // row_ror:4
    x = op(x, dpp_move<0x4E>(x));              // quad_perm [2,3,0,1]
    return op(x, dpp_move<0xB1>(x));           // quad_perm [1,0,3,2]
}

}  // namespace kavg
