// Pieces shared by the kernels that run all K local steps of a small fp32 model in one launch (fused_small.hip,
// fused_units.hip): tagged words for the exchange between workgroups, the counter-based index draw, reductions over
// the 16 lanes of a wavefront row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kavg {

// a partial and its tag as one 64-bit word
__device__ __forceinline__ void st_tagged(uint64_t* p, float v, uint32_t tag) {
    __hip_atomic_store(p, ((uint64_t)tag << 32) | __builtin_bit_cast(uint32_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_tagged(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// draw (learner, step, slot) of the index stream (the counter layout of index_stream_kernel)
__device__ __forceinline__ int32_t index_draw(uint64_t seed, uint32_t learner, uint32_t step, uint32_t slot, uint32_t N) {
    const uint64_t c = ((uint64_t)learner << 40) | ((uint64_t)step << 16) | slot;
    uint64_t z = seed + (c + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return (int32_t)((z ^ (z >> 31)) % (uint64_t)N);
}

// value of lane (l ^ pattern) within rows of 16 lanes, by data-parallel primitives (no LDS round trip)
template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// sum / maximum over each row of 16 lanes, left in all 16 (same operand pairs in every lane: bit-identical)
__device__ __forceinline__ float row16_sum(float x) {
    x += row_move<0xB1>(x);        // quad_perm [1,0,3,2]
    x += row_move<0x4E>(x);        // quad_perm [2,3,0,1]
    x += row_move<0x141>(x);       // row_half_mirror
    x += row_move<0x140>(x);       // row_mirror
    return x;
}
__device__ __forceinline__ float row16_max(float x) {
    x = fmaxf(x, row_move<0xB1>(x));
    x = fmaxf(x, row_move<0x4E>(x));
    x = fmaxf(x, row_move<0x141>(x));
    x = fmaxf(x, row_move<0x140>(x));
    return x;
}

}  // namespace kavg
