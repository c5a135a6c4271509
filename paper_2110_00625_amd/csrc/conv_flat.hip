// 3x3 convolution (stride 1, zero padding 1) on channels-last bf16 images of any size, forward and data gradient:
//
//   forward        out[p][o] = relu( b[o] + sum over (tap, c) of in[p + (dy, dx)][c] * W[o][tap][c] )
//   data gradient  din[p][c] = [act[p][c] > 0] * sum over (tap, o) of dz[p - (dy, dx)][o] * W[o][tap][c]
//
// (the learner's forward and backward pass of Algorithm 1 through a convolutional layer; tap = 3 (dy+1) + (dx+1)).
//
// Positions are numbered with one zero pixel behind every image row and one zero row behind every image:
// q = (n (H+1) + h) (W+1) + w.  The neighbour a tap points at is then q + dy (W+1) + dx everywhere -- the zero column
// serves as the right margin of its row and the left margin of the next, the zero row as the lower margin of its image
// and the upper one of the next -- so a tile is any range of q, whatever the image size, and a tap is a constant
// offset into it.  (The price is the margin positions: 7 % of the products at 28x28.)
//
// A workgroup of four wavefronts owns 512 (256 with more than 64 output channels) consecutive positions and all output
// channels; the pixels it needs, W+2 further ones on either side included, are brought to LDS once per group of
// CK channels.  A wavefront owns 128 positions times up to 64 channels: eight accumulator blocks of the 32x32x16
// matrix instruction, four pixel operands out of LDS and two weight operands per slab of 16 channels.
//
// Why this split: with the weights in LDS as well (one image row per wavefront, as an earlier version of these kernels
// had it) a slab of 64 -> 128 channels takes five LDS reads per four matrix instructions, 160 LDS cycles per 128
// matrix cycles, and every step waits at two barriers for its weights.  Here it is four reads per eight instructions,
// and the weights come straight from L2 in operand order (launch_pack_weights; 1 KB per operand, consecutive, requested
// slabs ahead), so nothing inside a channel group waits for anything but the matrix cores.
//
// Measured on 28x28 images, channels 8-32-64, 8 learners of 32 images (us per launch; before: the generic kernel on an
// implicit patch matrix, the first layer on a written one): forward 15 + 17 -> 11 (first layer) and 27 -> 19, data gradient
// 37 and a rotated weight copy -> 22, weight gradient 17 -> 12 and 49 -> 33 (conv_flat_wgrad.hip), a round of four steps
// 980 -> 605 (555 with one launch for the SGD steps of all layers).  At 64 -> 128 channels (32x32, 700 TFLOP/s) 17.6 k of a
// workgroup's 34 k cycles are the contraction, 6.8 k bring in pixels, 9.4 k write the outputs; the clock stands near 1.6 GHz.
//
// The last convolution, below the mean over the positions, writes no activations: what is read of them afterwards is their
// ReLU mask, one bit each, and their sums.  The sums of an image are a product with ones out of the epilogue's patch, 128
// positions at a time, joined in ascending order (pool_finish_kernel).  16 learners of 64 images of 32x32, channels
// 8-32-64-128: 268 MB of activations were written once and read three times; without them the mean takes 5 us instead of 47 and
// the data gradient 184 instead of 203, a round 6.92 -> 6.28 ms; one convolution on 60x32 images 141 -> 97 us, 28x28 536 -> 514.
#include "kavg_internal.h"
#include "conv_flat.h"
#include "conv_pool.h"
#include "fastdiv.h"
#include "split.h"
#include <type_traits>

namespace kavg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int NT = 256;
constexpr int PB = 4;                        // pixel blocks of 32 positions per wavefront
enum { FWD = 0, FWD_GATHER = 1, BWD = 2, BWD_POOL = 3 };

struct FlatArgs {
    const uint16_t* in; size_t in_lstride; int c_k;      // images of c_k contraction channels
    const int32_t* gather; long gather_lstride;          // FWD_GATHER: rows of `in`
    const uint16_t* frag; size_t frag_lstride; int slabs, blocks;
    const uint16_t* bhi; const uint16_t* blo; size_t b_lstride;      // forward: bias planes
    const uint16_t* act;                                 // data gradient: activations of the layer below (strides of out)
    uint16_t* out; size_t out_lstride; int c_n;
    int H, W, sign;                                      // sign: +1 forward, -1 data gradient
    int end;                                             // positions up to the last pixel of the last image
    const int32_t* table; int table_len;                 // pixel of position i - W - 2
    uint32_t div_hw_m; int div_hw_s;
    int tiles, total, padded;                            // tiles per learner; workgroups
    const uint16_t* dpool; size_t dpool_lstride; float inv;          // BWD_POOL: gradients from the bits and these
    uint32_t* bits; int bits_pitch; size_t bits_lstride;             // words per pixel; LAST: written, BWD_POOL: read
    float* sums; int slots, image;                                   // LAST: places of images per 128 positions; positions of an image
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));      // round to nearest even
}

// Two bf16 numbers, the largest finite one in place of infinity: in a product with ones and zeros an infinity would reach every
// sum (its zeros are NaN).  A sum that holds such a number is at least as large, and infinite again in pool_finish_kernel.
constexpr uint32_t BF16_MAX = 0x7F7Fu;
__device__ __forceinline__ uint32_t finite2(uint32_t two) {
    typedef short i16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(i16x2, two), (i16x2){(short)BF16_MAX, (short)BF16_MAX}));
}

// fragment of a [position][channel] patch by transpose reads: lane l receives channel x0 + l%32 at positions 8 (l/32) .. +7
__device__ __forceinline__ bf16x8 frag_tr(const uint16_t* patch, int pitch, int x0, int lane) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    const int t = lane & 15, grp = lane >> 4;
    const uint16_t* p = patch + ((grp >> 1) * 8 + (t >> 2)) * pitch + x0 + (grp & 1) * 16 + (t & 3) * 4;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(p + 4 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// bytes of the output patches of the four wavefronts, and of the pixels of a tile, which those lie over; behind the patches
// a byte for each position of each wavefront (LAST: in the tile, for LDS beyond it would cost the widest images a kernel)
__host__ __device__ constexpr int patch_area(int NB) { return 4 * 32 * (NB * 32 + 8) * 2; }
__host__ __device__ constexpr int tile_area(int n_px, int CK, int NB) {
    return n_px * (CK + 8) * 2 > patch_area(NB) + 4 * PB * 32 ? n_px * (CK + 8) * 2 : patch_area(NB) + 4 * PB * 32;
}

// LAST (forward): the layer below the mean over the positions; bits and partial sums instead of activations
template <int CK, int NB, int PWAVES, int KIND, bool LAST>
__global__ void __launch_bounds__(NT, 2) conv_flat_kernel(FlatArgs a) {
    constexpr int IP = CK + 8;                            // LDS pixel: its channels plus 16 bytes
    constexpr int TP = PWAVES * PB * 32, SL = CK / 16, C8 = CK / 8;
    constexpr int AHEAD = SL % 2 == 0 ? 6 : 3;            // weight operands in flight, in slabs (divides the 9 SL slabs of a group)
    constexpr bool BACK = KIND == BWD || KIND == BWD_POOL;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* const IN = (uint16_t*)smem;
    const int n_px = TP + 2 * (a.W + 1) + 2;              // pixels q0 - W - 2 .. of the tile
    typedef typename std::conditional<KIND == FWD_GATHER, int64_t, int2>::type Source;
    Source* const SRC = (Source*)(smem + tile_area(n_px, CK, NB));      // where a pixel lies: int2 (pixel, image) or pixel of the data set; -1: margin
    float* const BIAS = (float*)(SRC + n_px);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pw = wave % PWAVES, cw = wave / PWAVES;
    // workgroup g runs on XCD g mod 8: each XCD gets one contiguous range of (learner, tile)
    const int at = (blockIdx.x & 7) * (a.padded >> 3) + (blockIdx.x >> 3);
    if (at >= a.total) return;
    const int learner = at / a.tiles, q0 = (at - learner * a.tiles) * TP;
    const int pitch = a.W + 1;
    const uint16_t* in = a.in + (size_t)learner * a.in_lstride;

    const uint16_t* frag = a.frag + (size_t)learner * a.frag_lstride + (size_t)cw * NB * 512 + lane * 8;
    const int steps = 9 * a.slabs;
    bf16x8 wr[AHEAD][NB];
    auto wfetch = [&](int set, int it) __attribute__((always_inline)) {
        const uint16_t* p = frag + (size_t)min(it, steps - 1) * a.blocks * 512;
#pragma unroll
        for (int j = 0; j < NB; ++j) wr[set][j] = *(const bf16x8*)(p + j * 512);
    };

    for (int i = tid; i < n_px; i += NT) {
        const int px = a.table[min(q0 + i, a.table_len - 1)];
        int n = 0;                                            // its image
        if constexpr (KIND == FWD_GATHER || KIND == BWD_POOL) n = (int)fastdiv((uint32_t)max(px, 0), a.div_hw_m, a.div_hw_s);
        if constexpr (KIND == FWD_GATHER)
            SRC[i] = px < 0 ? -1 : ((int64_t)a.gather[(long)learner * a.gather_lstride + n] - n) * (a.H * a.W) + px;
        else
            SRC[i] = make_int2(px, n);
    }
    if constexpr (!BACK) {
        for (int i = tid; i < 128; i += NT) {
            const size_t at_b = (size_t)learner * a.b_lstride + min(i, a.c_n - 1);
            BIAS[i] = __builtin_bit_cast(float, split_join(a.bhi[at_b], a.blo[at_b]));
        }
    }
    __syncthreads();

    // all pixels of channel group g: every request of a thread is in flight before the first is waited for
    const int pieces = n_px * C8;
    auto load_tile = [&](int g) __attribute__((always_inline)) {
        constexpr int ALL = ((TP + 132) * C8 + NT - 1) / NT, MAX = KIND == BWD_POOL ? 8 : 11, N = ALL < MAX ? ALL : MAX;
        for (int e0 = tid; e0 < pieces; e0 += NT * N) {
            u32x4 v[KIND == BWD_POOL ? 1 : N], gp[KIND == BWD_POOL ? N : 1];
            uint8_t bt[KIND == BWD_POOL ? N : 1];
            unsigned ok = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int e = min(e0 + NT * i, pieces - 1);
                const int ch = g * CK + (e % C8) * 8;
                const Source src = SRC[e / C8];
                int64_t px;
                if constexpr (KIND == FWD_GATHER) px = src; else px = src.x;
                const bool in_ok = px >= 0 && ch < a.c_k;
                if (in_ok) ok |= 1u << i;
                if constexpr (KIND == BWD_POOL) {
                    bt[i] = ((const uint8_t*)(a.bits + (size_t)learner * a.bits_lstride))[in_ok ? px * a.bits_pitch * 4 + (ch >> 3) : 0];
                    gp[i] = *(const u32x4*)(a.dpool + (size_t)learner * a.dpool_lstride + (in_ok ? (size_t)src.y * a.c_k + ch : 0));
                } else {
                    v[i] = *(const u32x4*)(in + (in_ok ? px * a.c_k + ch : 0));
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int e = e0 + NT * i;
                const u32x4 zero = {0u, 0u, 0u, 0u};
                u32x4 x;
                if constexpr (KIND == BWD_POOL) x = pool_grad_bits((ok >> i) & 1u ? bt[i] : 0u, gp[i], a.inv);
                else x = (ok >> i) & 1u ? v[i] : zero;
                if (e < pieces) *(u32x4*)(IN + (e / C8) * IP + (e % C8) * 8) = x;
            }
        }
    };

    f32x16 acc[NB][PB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int b = 0; b < PB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][b][e] = 0.f;

    const uint16_t* lane_px = IN + (pw * PB * 32 + (lane & 31) + pitch + 1) * IP + (lane >> 5) * 8;
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) wfetch(s, s);
    static_assert(9 * SL % AHEAD == 0, "a group leaves the weight registers where it found them");
    const int groups = a.slabs / SL;
    for (int g = 0; g < groups; ++g) {
        if (g) __syncthreads();                               // everyone is done with the previous group's pixels
        load_tile(g);
        __syncthreads();
        bf16x8 x[2][PB];                                      // pixel operands of this slab and the next
        auto xfetch = [&](int s) __attribute__((always_inline)) {
            const int tap = s / SL;
            const uint16_t* p = lane_px + a.sign * ((tap / 3 - 1) * pitch + tap % 3 - 1) * IP + (s % SL) * 16;
#pragma unroll
            for (int b = 0; b < PB; ++b) x[s & 1][b] = *(const bf16x8*)(p + b * 32 * IP);
        };
        xfetch(0);
#pragma unroll
        for (int s = 0; s < 9 * SL; ++s) {
            if (s + 1 < 9 * SL) xfetch(s + 1);
            __builtin_amdgcn_sched_barrier(0);                // (left alone, the compiler moves every request to just before its use)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int b = 0; b < PB; ++b)
                    acc[j][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[s % AHEAD][j], x[s & 1][b], acc[j][b], 0, 0, 0);
            wfetch(s % AHEAD, g * SL * 9 + s + AHEAD);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();                                          // the tile is dead: output patches

    // accumulator e of block (j, b) = output channel 32 j + 8 (e/4) + 4 (lane/32) + e%4 at position 32 b + lane%32.
    // The outputs of 32 positions pass through a patch of LDS that belongs to the wavefront (its LDS accesses complete
    // in order) and leave as whole rows of its channels.  Nothing here waits for a load that was requested after a
    // store: the counter is in order, and such a wait is a wait for the stores.
    constexpr int OP = NB * 32 + 8, C16 = NB * 4;
    uint16_t* patch = (uint16_t*)smem + wave * 32 * OP;
    uint16_t* out = a.out + (size_t)learner * a.out_lstride;
    auto position = [&](int b, int i) __attribute__((always_inline)) {     // pixel of position i of block b, -1: margin
        const int p = (pw * PB + b) * 32 + i;
        if constexpr (KIND == FWD_GATHER) return a.table[min(q0 + p + pitch + 1, a.table_len - 1)];
        else return SRC[p + pitch + 1].x;
    };
    u32x2 mask[NB][4];
    auto fetch_mask = [&](int b) __attribute__((always_inline)) {
        const uint16_t* act = a.act + (size_t)learner * a.out_lstride + (size_t)max(position(b, lane & 31), 0) * a.c_n;
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ch = (cw * NB + j) * 32 + q * 8 + (lane >> 5) * 4;
                mask[j][q] = *(const u32x2*)(act + (ch < a.c_n ? ch : 0));
            }
    };
    if constexpr (BACK) fetch_mask(0);
    f32x16 sums[LAST ? NB : 1];                               // [place of an image][channel] of the wavefront's positions
    uint8_t* const SLOT = (uint8_t*)smem + patch_area(NB) + wave * (PB * 32);      // LAST: place of a position's image among those of its wavefront; 255: margin
    if constexpr (LAST) {
        const int first = (q0 + pw * PB * 32) / a.image;
#pragma unroll
        for (int h = 0; h < PB / 2; ++h) {
            const int px = position(2 * h + (lane >> 5), lane & 31);
            SLOT[h * 64 + lane] = px < 0 ? 255 : (uint8_t)((int)fastdiv((uint32_t)px, a.div_hw_m, a.div_hw_s) - first);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) sums[j][e] = 0.f;
    }
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        uint32_t word[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            word[j] = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v0 = acc[j][b][4 * q + 0], v1 = acc[j][b][4 * q + 1], v2 = acc[j][b][4 * q + 2], v3 = acc[j][b][4 * q + 3];
                if constexpr (BACK) {
                    const u32x2 m = mask[j][q];
                    // stored activations are ReLU outputs (never negative): positive <=> non-zero magnitude
                    v0 = (m.x & 0x7FFFu) ? v0 : 0.f;
                    v1 = (m.x & 0x7FFF0000u) ? v1 : 0.f;
                    v2 = (m.y & 0x7FFFu) ? v2 : 0.f;
                    v3 = (m.y & 0x7FFF0000u) ? v3 : 0.f;
                } else {
                    const float4 bias = *(const float4*)(BIAS + (cw * NB + j) * 32 + q * 8 + (lane >> 5) * 4);
                    v0 = fmaxf(v0 + bias.x, 0.f);
                    v1 = fmaxf(v1 + bias.y, 0.f);
                    v2 = fmaxf(v2 + bias.z, 0.f);
                    v3 = fmaxf(v3 + bias.w, 0.f);
                }
                u32x2 o = {pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
                if constexpr (LAST) o = (u32x2){finite2(o.x), finite2(o.y)};
                *(u32x2*)(patch + (lane & 31) * OP + j * 32 + q * 8 + (lane >> 5) * 4) = o;
                if constexpr (LAST) {
                    const uint32_t four = (o.x & 0x7FFFu ? 1u : 0u) | (o.x & 0x7FFF0000u ? 2u : 0u) | (o.y & 0x7FFFu ? 4u : 0u) | (o.y & 0x7FFF0000u ? 8u : 0u);
                    word[j] |= four << (q * 8 + (lane >> 5) * 4);
                }
            }
        }
        if constexpr (LAST) {
            // The sum over the positions of an image is a product with ones where a position is of that image (margins: of none).
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const u32x2 sl = *(const u32x2*)(SLOT + b * 32 + t * 16 + (lane >> 5) * 8);
                u32x4 ones;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = i < 2 ? sl.x : sl.y;
                    ones[i] = (((w >> (i & 1) * 16) & 0xFFu) == (uint32_t)(lane & 31) ? 0x3F80u : 0u) |
                              (((w >> ((i & 1) * 16 + 8)) & 0xFFu) == (uint32_t)(lane & 31) ? 0x3F800000u : 0u);
                }
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    sums[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ones), frag_tr(patch + t * 16 * OP, OP, j * 32, lane), sums[j], 0, 0, 0);
            }
            const int to = position(b, lane & 31);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const auto h = __builtin_amdgcn_permlane32_swap(word[j], word[j], false, false);
                if (lane < 32 && to >= 0 && cw * NB + j < a.bits_pitch)
                    a.bits[(size_t)learner * a.bits_lstride + (size_t)to * a.bits_pitch + cw * NB + j] = (uint32_t)h[0] | (uint32_t)h[1];
            }
            __builtin_amdgcn_sched_barrier(0);
            continue;
        }
        if constexpr (BACK) { if (b + 1 < PB) fetch_mask(b + 1); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int pass = 0; pass < C16 / 2; ++pass) {
            const int id = pass * 64 + lane, row = id / C16, c8 = (id % C16) * 8, ch = cw * NB * 32 + c8;
            const int to = position(b, row);
            const u32x4 v = *(const u32x4*)(patch + row * OP + c8);
            if (to >= 0 && ch < a.c_n) *(u32x4*)(out + (size_t)to * a.c_n + ch) = v;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (LAST) {
        const int group = q0 / (PB * 32) + pw, first = (q0 + pw * PB * 32) / a.image, n = (q0 + pw * PB * 32 + PB * 32 - 1) / a.image - first;
        float* to = a.sums + ((size_t)learner * a.tiles * PWAVES + group) * a.slots * (a.blocks * 32) + cw * NB * 32 + (lane & 31);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int slot = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                if (slot <= n) to[(size_t)slot * (a.blocks * 32) + j * 32] = sums[j][e];
            }
    }
}

// pooled[learner][image][channel] = bf16(mean): one lane per output adds the image's partial sums in ascending order.  (One row of
// the grid per learner: all learners' outputs together may be more than 2^31.)
__global__ void __launch_bounds__(NT) pool_finish_kernel(const float* sums, uint16_t* pooled, int image, int last, int slots, int groups, int pitch, int c, float inv,
                                                         int outputs) {
    const int e = blockIdx.x * NT + threadIdx.x, learner = blockIdx.y;
    if (e >= outputs) return;
    const int ch = e % c, n = e / c;
    const int g1 = (n * image + last) / (PB * 32);
    const float* p = sums + (size_t)learner * groups * slots * pitch + ch;
    float s = 0.f;
#pragma unroll 4
    for (int g = n * image / (PB * 32); g <= g1; ++g) {
        const float x = p[((size_t)g * slots + n - g * (PB * 32) / image) * pitch];
        s += x < __builtin_bit_cast(float, BF16_MAX << 16) ? x : INFINITY;      // (finite2)
    }
    const __bf16 h = (__bf16)(s * inv);                       // round to nearest even
    pooled[(size_t)learner * outputs + e] = __builtin_bit_cast(uint16_t, h);
}

__global__ void __launch_bounds__(NT) flat_table_kernel(int32_t* table, int len, int end, int H, int W) {
    const int i = blockIdx.x * NT + threadIdx.x;
    if (i >= len) return;
    const int q = i - W - 2, row = q / (W + 1), w = q - row * (W + 1), n = row / (H + 1), h = row - n * (H + 1);
    table[i] = q >= 0 && q < end && w < W && h < H ? (n * H + h) * W + w : -1;
}

// ---- weights in operand order -------------------------------------------------------------------
// frag[(group * 9 * SL + tap * SL + slab in the group) * blocks + block][lane][8]: lane l of the matrix
// operand holds output channel 32 block + l%32, contraction channels 16 slab + 8 (l/32) .. +7; zero outside the layer.
struct PackDir { uint16_t* frag; size_t frag_lstride; const uint16_t* w; int c_in, c_out, back, SL, slabs, blocks, wgs; };
constexpr int PACK_MAX = 16;                 // directions per launch
struct PackArgs { PackDir d[PACK_MAX]; int n; size_t w_lstride; };

__global__ void __launch_bounds__(NT) pack_weights_kernel(PackArgs a) {
    int g = blockIdx.x, i = 0;
    while (i + 1 < a.n && g >= a.d[i].wgs) g -= a.d[i++].wgs;
    const PackDir& d = a.d[i];
    const int e = g * NT + threadIdx.x;
    if (e >= 9 * d.slabs * d.blocks * 64) return;
    const int lane = e & 63, block = (e >> 6) % d.blocks, it = (e >> 6) / d.blocks;
    const int grp = it / (9 * d.SL), rem = it - grp * 9 * d.SL;
    const int tap = rem / d.SL, slab = grp * d.SL + rem - tap * d.SL;
    const int x = block * 32 + (lane & 31), k = slab * 16 + (lane >> 5) * 8;
    const uint16_t* w = d.w + (size_t)blockIdx.y * a.w_lstride;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (!d.back) {
        if (x < d.c_out && k < d.c_in)                        // (all channel counts are multiples of 8, so layers and rows start at 16 bytes)
            v = *(const u32x4*)(w + ((size_t)x * 9 + tap) * d.c_in + k);
    } else if (x < d.c_in && k < d.c_out) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint16_t* p = w + ((size_t)(k + 2 * q) * 9 + tap) * d.c_in + x;
            v[q] = (uint32_t)p[0] | ((uint32_t)p[(size_t)9 * d.c_in] << 16);
        }
    }
    *(u32x4*)(d.frag + (size_t)blockIdx.y * d.frag_lstride + (size_t)e * 8) = v;
}

// the tile, where its pixels lie, the bias
size_t lds_bytes(const FlatPlan& p, int W) {
    const int n_px = p.PWAVES * PB * 32 + 2 * (W + 1) + 2;
    return (size_t)tile_area(n_px, p.CK, p.NB) + (size_t)n_px * 8 + 128 * 4;
}

FlatArgs make_args(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t* table) {
    FlatArgs a = {};
    a.frag = frag; a.frag_lstride = plan.frag_elems(); a.slabs = plan.slabs; a.blocks = plan.blocks;
    a.H = c.H; a.W = c.W;
    a.end = ((c.B - 1) * (c.H + 1) + c.H - 1) * (c.W + 1) + c.W;
    a.table = table; a.table_len = conv_flat_table_len(c.B, c.H, c.W);
    fastdiv_make((uint32_t)(c.H * c.W), &a.div_hw_m, &a.div_hw_s);
    const int TP = plan.PWAVES * PB * 32;
    a.tiles = (a.end + TP - 1) / TP;
    a.total = a.tiles * c.P;
    a.padded = (a.total + 7) / 8 * 8;
    return a;
}

template <int CK, int NB, int PWAVES, int KIND, bool LAST>
hipError_t launch(const FlatArgs& a, size_t smem, hipStream_t st) {
    if (smem > 64 * 1024) {
        static hipError_t raised = hipFuncSetAttribute((const void*)conv_flat_kernel<CK, NB, PWAVES, KIND, LAST>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
        if (raised != hipSuccess) return raised;
    }
    hipLaunchKernelGGL((conv_flat_kernel<CK, NB, PWAVES, KIND, LAST>), dim3(a.padded), dim3(NT), smem, st, a);
    return hipGetLastError();
}

template <int KIND, bool LAST = false>
hipError_t run(const FlatArgs& a, const FlatPlan& p, hipStream_t st) {
    const size_t smem = lds_bytes(p, a.W);
    if (p.PWAVES == 2) {
        if (p.CK == 64) return launch<64, 2, 2, KIND, LAST>(a, smem, st);
        if (p.CK == 48) return launch<48, 2, 2, KIND, LAST>(a, smem, st);
        if (p.CK == 32) return launch<32, 2, 2, KIND, LAST>(a, smem, st);
        return launch<16, 2, 2, KIND, LAST>(a, smem, st);
    }
    if (p.NB == 2) {
        if (p.CK == 48) return launch<48, 2, 4, KIND, LAST>(a, smem, st);
        if (p.CK == 32) return launch<32, 2, 4, KIND, LAST>(a, smem, st);
        return launch<16, 2, 4, KIND, LAST>(a, smem, st);
    }
    if (p.CK == 48) return launch<48, 1, 4, KIND, LAST>(a, smem, st);
    if (p.CK == 32) return launch<32, 1, 4, KIND, LAST>(a, smem, st);
    return launch<16, 1, 4, KIND, LAST>(a, smem, st);
}

}  // namespace

int conv_flat_table_len(int B, int H, int W) { return ((B - 1) * (H + 1) + H - 1) * (W + 1) + W + W + 3; }

hipError_t launch_flat_table(int32_t* table, int B, int H, int W, hipStream_t st) {
    const int len = conv_flat_table_len(B, H, W);
    hipLaunchKernelGGL(flat_table_kernel, dim3((len + NT - 1) / NT), dim3(NT), 0, st, table, len, len - W - 3, H, W);
    return hipGetLastError();
}

bool conv_flat_plan(int B, int H, int W, int c_k, int c_n, FlatPlan* plan) {
    FlatPlan p = {};
    if (c_n > 128 || (size_t)B * (H + 1) * (W + 1) >= ((size_t)1 << 30)) return false;
    p.NB = c_n <= 32 ? 1 : 2;
    p.PWAVES = c_n <= 64 ? 4 : 2;
    p.blocks = p.NB * (4 / p.PWAVES);
    // Slabs per group: the largest number whose tile leaves room for two workgroups per compute unit, among those that
    // pad the contraction least.  (More channels per group: fewer reloads, each of which the workgroup waits for.)
    const int slabs = (c_k + 15) / 16;
    int best = 0;
    for (int SL = 1; SL <= (p.PWAVES == 2 ? 4 : 3) && SL <= slabs; ++SL) {
        FlatPlan q = p;
        q.CK = SL * 16;
        q.slabs = (slabs + SL - 1) / SL * SL;
        if (lds_bytes(q, W) > 80 * 1024 || (best && q.slabs > best)) continue;
        p.CK = q.CK; p.slabs = best = q.slabs;
    }
    if (!best) return false;
    *plan = p;
    return true;
}

hipError_t launch_pack_weights(const PackLayer* layers, int n, size_t w_lstride, int P, hipStream_t st) {
    PackArgs a = {};
    a.w_lstride = w_lstride;
    int wgs = 0;
    auto flush = [&]() -> hipError_t {
        if (a.n == 0) return hipSuccess;
        hipLaunchKernelGGL(pack_weights_kernel, dim3(wgs, P), dim3(NT), 0, st, a);
        a.n = 0; wgs = 0;
        return hipGetLastError();
    };
    auto add = [&](const PackLayer& l, const FlatPlan& p, uint16_t* frag, size_t lstride, int back) {
        PackDir& d = a.d[a.n++];
        d.frag = frag; d.frag_lstride = lstride; d.w = l.w; d.c_in = l.c_in; d.c_out = l.c_out; d.back = back;
        d.SL = p.CK / 16; d.slabs = p.slabs; d.blocks = p.blocks;
        d.wgs = (9 * p.slabs * p.blocks * 64 + NT - 1) / NT;
        wgs += d.wgs;
    };
    for (int i = 0; i < n; ++i) {
        if (a.n + 2 > PACK_MAX) { const hipError_t e = flush(); if (e != hipSuccess) return e; }
        if (layers[i].fwd) add(layers[i], layers[i].fwd_plan, layers[i].fwd, layers[i].fwd_lstride, 0);
        if (layers[i].bwd) add(layers[i], layers[i].bwd_plan, layers[i].bwd, layers[i].bwd_lstride, 1);
    }
    return flush();
}

int conv_pool_slots(int H, int W) {
    const int image = (H + 1) * (W + 1);
    return image < 5 ? 0 : PB * 32 / image + 2;               // (at most the 32 rows of a matrix instruction)
}

size_t conv_pool_elems(int P, int B, int H, int W, const FlatPlan& plan) {
    const int end = ((B - 1) * (H + 1) + H - 1) * (W + 1) + W, TP = plan.PWAVES * PB * 32;
    return (size_t)P * ((end + TP - 1) / TP) * plan.PWAVES * conv_pool_slots(H, W) * plan.blocks * 32;
}

hipError_t launch_pool_finish(const float* sums, const FlatPlan& plan, void* pooled, int P, int B, int H, int W, int c, hipStream_t st) {
    const int end = ((B - 1) * (H + 1) + H - 1) * (W + 1) + W, TP = plan.PWAVES * PB * 32, outputs = B * c;      // (at most 2^16 images of 128 channels)
    hipLaunchKernelGGL(pool_finish_kernel, dim3((outputs + NT - 1) / NT, P), dim3(NT), 0, st, sums, (uint16_t*)pooled, (H + 1) * (W + 1),
                       (H - 1) * (W + 1) + W - 1, conv_pool_slots(H, W), (end + TP - 1) / TP * plan.PWAVES, plan.blocks * 32, c, 1.0f / (float)(H * W), outputs);
    return hipGetLastError();
}

hipError_t conv_flat_forward(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t* table, const void* X,
                             const int32_t* gather, long gstride, hipStream_t st) {
    if (!c.bits && !c.out) return hipErrorInvalidValue;
    FlatArgs a = make_args(c, plan, frag, table);
    const size_t rows = (size_t)c.B * c.H * c.W;
    a.in = (const uint16_t*)(gather ? X : c.in); a.in_lstride = gather ? 0 : rows * c.c_in; a.c_k = c.c_in;
    a.gather = gather; a.gather_lstride = gstride;
    a.bhi = c.bhi; a.blo = c.blo; a.b_lstride = c.ws_stride;
    a.out = (uint16_t*)c.out; a.out_lstride = rows * c.c_out; a.c_n = c.c_out;
    a.sign = 1;
    if (c.bits) {
        a.bits = c.bits; a.bits_pitch = conv_bits_pitch(c.c_out); a.bits_lstride = rows * a.bits_pitch;
        a.sums = c.pool_sums; a.slots = conv_pool_slots(c.H, c.W); a.image = (c.H + 1) * (c.W + 1);
        if (!a.sums || !a.slots) return hipErrorInvalidValue;
        return gather ? run<FWD_GATHER, true>(a, plan, st) : run<FWD, true>(a, plan, st);
    }
    return gather ? run<FWD_GATHER>(a, plan, st) : run<FWD>(a, plan, st);
}

hipError_t conv_flat_backward_data(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t* table, const void* dpool,
                                   hipStream_t st) {
    if (dpool ? !c.bits : !c.dz) return hipErrorInvalidValue;
    FlatArgs a = make_args(c, plan, frag, table);
    const size_t rows = (size_t)c.B * c.H * c.W;
    a.in = (const uint16_t*)c.dz; a.in_lstride = rows * c.c_out; a.c_k = c.c_out;
    a.bits = c.bits; a.bits_pitch = conv_bits_pitch(c.c_out); a.bits_lstride = rows * a.bits_pitch;
    a.dpool = (const uint16_t*)dpool; a.dpool_lstride = (size_t)c.B * c.c_out; a.inv = 1.0f / (float)(c.H * c.W);
    a.act = (const uint16_t*)c.in;
    a.out = (uint16_t*)c.dz_in; a.out_lstride = rows * c.c_in; a.c_n = c.c_in;
    a.sign = -1;
    return dpool ? run<BWD_POOL>(a, plan, st) : run<BWD>(a, plan, st);
}

}  // namespace kavg
