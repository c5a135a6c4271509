// Column sums of dZ (bias gradients) beside the products that use it, every column one fp32 chain over ascending samples.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kavg {

// Adds a slab of 16 samples to the chain s of unit lane%32: z holds samples 8 (lane/32) .. +7 of the slab (the operand of the
// matrix instruction as it lies in registers).  Both halves of the wavefront add all the time; the half that holds the next
// samples is the one whose sum counts, and hands it to the other.  Eight of these are dependent additions, no LDS access: summed
// from LDS a tile with a bias took half a microsecond longer per 64 samples.
template <class Z>
__device__ __forceinline__ float column_sum16(const Z& z, float s) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 w = __builtin_bit_cast(u32x4, z);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s += __builtin_bit_cast(float, w[i] << 16);
            s += __builtin_bit_cast(float, w[i] & 0xFFFF0000u);
        }
        const uint32_t b = __builtin_bit_cast(uint32_t, s);
        const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);   // [0]: the lower half's values in both, [1]: the upper's
        s = __builtin_bit_cast(float, (uint32_t)r[half]);
    }
    return s;
}

}  // namespace kavg
