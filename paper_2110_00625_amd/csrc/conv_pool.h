// Gradient of the mean over the positions, eight channels at a time: what the layer above hands the last
// convolution is dpool[image][channel]; the gradient w.r.t. that convolution's pre-activation at a position is
// bf16( [act > 0] * dpool / (H W) ).  Used by pool_backward_kernel and by the kernels that form these values
// while loading, instead of reading them from a buffer.
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <type_traits>

namespace kavg {

typedef uint32_t pool_u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pool_pack2(float lo, float hi) {
    const __bf16 a = (__bf16)lo, b = (__bf16)hi;          // round to nearest even
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

// ones in the halves of `two` that are not +-0 (stored activations are ReLU outputs, never negative: positive <=> non-zero magnitude)
__device__ __forceinline__ uint32_t where_nonzero2(uint32_t two) {
    typedef short i16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, (two & 0x7FFF7FFFu) + 0x7FFF7FFFu) >> (i16x2){15, 15});
}

// m: eight activations (ReLU outputs, bf16 pairs); g: the eight channels' dpool; inv = 1 / (H W)
__device__ __forceinline__ pool_u32x4 pool_grad_piece(pool_u32x4 m, pool_u32x4 g, float inv) {
    pool_u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float g0 = __builtin_bit_cast(float, g[q] << 16) * inv, g1 = __builtin_bit_cast(float, g[q] & 0xFFFF0000u) * inv;
        // stored activations are never negative: positive <=> non-zero magnitude
        o[q] = pool_pack2((m[q] & 0x7FFFu) ? g0 : 0.f, (m[q] & 0x7FFF0000u) ? g1 : 0.f);
    }
    return o;
}

// The same in two parts, for kernels that scale a channel's gradient once and mask it at every position: bf16(g / (H W)) ...
__device__ __forceinline__ pool_u32x4 pool_scale(pool_u32x4 g, float inv) {
    pool_u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = pool_pack2(__builtin_bit_cast(float, g[q] << 16) * inv, __builtin_bit_cast(float, g[q] & 0xFFFF0000u) * inv);
    return o;
}

// ... and eight of those where the bits that the last convolution's forward pass leaves in place of its activations are set (bit c
// of m: channel c of the eight is positive; ConvCall::bits).  16 instructions; scaled and rounded at every position it was 45,
// more than half of what the weight gradient's wavefronts did beside their products.
__device__ __forceinline__ pool_u32x4 pool_mask(uint32_t m, pool_u32x4 scaled) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        scaled[q] &= ((uint32_t)__builtin_amdgcn_sbfe((int)m, 2 * q, 1) & 0xFFFFu) | ((uint32_t)__builtin_amdgcn_sbfe((int)m, 2 * q + 1, 1) & 0xFFFF0000u);
    return scaled;
}
__device__ __forceinline__ pool_u32x4 pool_grad_bits(uint32_t m, pool_u32x4 g, float inv) { return pool_mask(m, pool_scale(g, inv)); }


// The mean over the positions from the partial sums that the last convolution's forward pass leaves (conv_flat.hip): places of images, of
// `pitch` channels each, per `group` positions.
struct PoolSums { const float* sums; int image, last, slots, group, groups, pitch; float inv; };

// ... of channel ch of image n, bf16: the partial sums in ascending order, the first four and then sixteen or eight on their way.  (A
// sum that holds the largest finite number stands for an infinity, see conv_flat.hip.)  Latency bounds it: four at a time it was 64 waits for
// an image of 127x128, of 256 partial sums.  (us per round of four steps, four at a time / so: 127x128, channels 8-128, one learner of one
// image 265 / 172, 100x100, 8-8, 2 of 1 202 / 141, 64x64, 8-16-128, 8 of 16 872 / 861; 28x28, 8-32-64, 8 of 32 410 / 412; with eight instead of the
// first four, images of few partial sums wait longer: 14x6, 8-128, 8 of 16, five steps 187 / 192.)
__device__ __forceinline__ uint16_t pool_mean(const PoolSums& q, int learner, int n, int ch) {
    const int g0 = n * q.image / q.group, g1 = (n * q.image + q.last) / q.group;
    const float* p = q.sums + ((size_t)learner * q.groups + g0) * q.slots * q.pitch + ch;
    const size_t step = (size_t)q.slots * q.pitch;
    // (the positions of the groups behind the first begin in this image: their first place.  Places beyond the last are read from there,
    // and not used)
    const size_t first = (size_t)(n - g0 * q.group / q.image) * q.pitch;
    const int m = g1 - g0;
    float s = 0.f;
    int g = 0;
    auto batch = [&](auto count) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        float x[N];
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = p[g + i == 0 ? first : min(g + i, m) * step];
#pragma unroll
        for (int i = 0; i < N; ++i) if (g + i <= m) s += x[i] < 0x1.FEp127f ? x[i] : __builtin_inff();
        g += N;
    };
    batch(std::integral_constant<int, 4>());
    while (m - g >= 8) batch(std::integral_constant<int, 16>());
    while (g <= m) batch(std::integral_constant<int, 8>());
    const __bf16 h = (__bf16)(s * q.inv);                     // round to nearest even
    return __builtin_bit_cast(uint16_t, h);
}

}  // namespace kavg
